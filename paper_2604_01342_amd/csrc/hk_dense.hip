// Dense dL/dalpha of the shared-decay large-M path (first term of eq. 9): the
// sum over events i of beta w_i K(t_i^-) into row m_i.
//
// The chunk is cut into blocks of 2^BL events (64 to 1024).  With tau_b
// the time of the event before block b, K_b the state there, and
//   c_i = beta w_i e^{-beta (t_i - tau_b)},   b_j = e^{beta (t_j - tau_b)},
// event i of block b adds c_i K_b to row m_i, and c_i b_j at (m_i, m_j) for
// the block's events j before it:
//   dense_prep    a workgroup per segment: the rows of K_b and of
//                 U_b[p] = sum of c_i over the block's events of node p
//                 the block's pair records (mark, place in the block, b_j) and
//                 the events' own records (c_i, w_i and the compensator term)
//                 partitioned by blocks of 16 nodes
//   dense_tiles   a workgroup per (block of 16 rows, event range), its tile of
//                 rows in float64 LDS.  Twelve waves add the pair terms (and
//                 sum w_i, for dL/dmu, and the compensator terms per node),
//                 four multiply U^T K over the range's blocks on the matrix
//                 cores: the pair terms are bound by LDS adds, the product by
//                 the matrix cores, and on one CU the two run side by side
// Why blocks: pair work grows with the block length (an own event meets half a
// block of records: 64-lane LDS atomics), the product with its inverse
// (M^2 multiply-adds per block), so the block length follows M.  Up to 1024
// nodes a tile holds whole rows: an own event is visited once, and every record
// lane of a visit but the last group's adds.  Beyond, a tile holds a block of
// columns, an own event is visited once for each, and meets that block's
// records only (a list per block of events and column block), so that blocks of
// events can grow with the column blocks.
// Measured per chunk of 2^20 events at M = 1000: dense_prep 32 us and
// dense_tiles 158 us (at equal issue priority of its waves 171, of which the
// pair terms alone 116 and the product alone, with the pair waves' loads,
// 124), against 27 + 304 us (and 12 for the partition's scatter, now in
// dense_prep) for tiles of 32 x 256 nodes walking windows of 128 column
// records; pair terms and product as two kernels: 120 + 89 us.  M = 4096, 1e6
// events: 710 us; 1999 with blocks of 256 events all of whose records every
// column block read, 1260 for the windows.
#include "hk_device.h"
#include "hk_large.h"
#include "hk_stream.h"
#include <type_traits>

namespace hk {

// inclusive sum of v over the lanes up to this one
__device__ __forceinline__ int32_t lane_incl_sum(int32_t v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t u = __shfl_up(v, d, 64);
        if (lane >= d) v += u;
    }
    return v;
}

// Workgroup s: the segment's 1024 events, wave v its events 256 v .. 256 v +
// 255 (a lane takes one event of each batch of 64).  The own records' places
// come from the counting sort of the partition (hk_bucket.hip): boff holds the
// starts of every (node block, segment) run, here each wave counts its events
// per node block and ranks them inside a batch by bit-sliced ballots.
// The pair records of a batch are permuted over the lanes by LDS bank: the
// pair kernel adds one own event's terms at the records' columns of one tile
// row with one LDS atomic, and the LDS serves 16 lanes of 8-byte words a
// cycle from 16 banks (column mod 16), so records sorted by bank and dealt
// round-robin over the four quarter-waves share a bank in a quarter only when
// more than four of the batch have it.  Nothing depends on the order: a record
// carries its place in the block.
// ML (several column blocks): a block's records are kept by column block, so that
// a workgroup of the pair kernel reads those of its own columns only: the same
// counting sort, into an LDS stage of whole groups of 64 (the rest of a list's
// last group empty), whose groups are then permuted as above and written out.
// LDS (dynamic): K and U as float64 [M], ML: the stage, then the partition's
// counters [4 + 1][NBO], ML: those of the lists and the blocks' groups.  Float64
// sums: LDS float32 atomics are far slower here.
// The rows are float32 where the product runs on the float32 matrix cores
// (large M), else float64.
// A lane of the product takes 16 bytes of a row of K, one column each of 4 (2)
// consecutive tiles of 16 columns: inside a group of 64 (32) columns the row is
// stored column-of-tile major.
template <typename RT>
__device__ __forceinline__ int32_t krow_at(int32_t q) {
    constexpr int V = 16 / sizeof(RT);   // tiles of 16 columns per group
    return (q & ~(16 * V - 1)) | ((q & 15) * V) | ((q >> 4) & (V - 1));
}
#define HK_PW 4   // waves per segment
// rank of this lane in (bank, lane) order, empty records last, dealt round-robin
// over the quarter-waves: a permutation of 0..63
__device__ __forceinline__ int bank_place(int bank, uint64_t lt) {
    uint64_t eq = ~0ull;
    int less = 0;
#pragma unroll
    for (int bit = 4; bit >= 0; --bit) {
        const uint64_t bi = __ballot((bank >> bit) & 1);
        const bool one = (bank >> bit) & 1;
        if (one) less += __builtin_popcountll(eq & ~bi);
        eq &= one ? bi : ~bi;
    }
    const int sidx = less + __builtin_popcountll(eq & lt);
    return (sidx & 3) * 16 + (sidx >> 2);
}
// the lanes of `valid` whose number of nbits bits is this lane's
__device__ __forceinline__ uint64_t same_number(uint64_t valid, int v, int nbits) {
    for (int bit = 0; bit < nbits; ++bit) {
        const uint64_t on = __ballot((v >> bit) & 1);
        valid &= ((v >> bit) & 1) ? on : ~on;
    }
    return valid;
}

template <int BL, typename RT, bool ML>
__global__ __launch_bounds__(64 * HK_PW) void dense_prep(int64_t c0, int32_t nev, int32_t M, int32_t Mp, int32_t NBO,
                                                         int32_t nbits, int32_t bs, double T,
                                                         const double* __restrict__ t,
                                                         const int32_t* __restrict__ marks,
                                                         const float* __restrict__ wchunk,
                                                         const float* __restrict__ beta,
                                                         const double* __restrict__ carry_seg,
                                                         const double* __restrict__ gcarry,
                                                         const double* __restrict__ seg_offdec, int32_t nseg,
                                                         const int32_t* __restrict__ boff,
                                                         int32_t* __restrict__ bbase, uint32_t* __restrict__ bo_key,
                                                         float2* __restrict__ bo_cw, double* __restrict__ bo_e,
                                                         uint2* __restrict__ prec, int32_t* __restrict__ wide,
                                                         RT* __restrict__ urow, RT* __restrict__ krow, int32_t rep,
                                                         int32_t CW, int32_t NCB, int32_t cbits,
                                                         int32_t* __restrict__ plist) {
    constexpr int NBK = HK_SEG >> BL;            // blocks per segment
    constexpr int NBT = HK_SEG / 64 / HK_PW;     // batches per wave
    static_assert(NBT * 64 * HK_PW == HK_SEG && BL >= 6 && BL <= 10,
                  "whole batches per wave, whole blocks per segment");
    extern __shared__ double lds[];
    double* Kl = lds;
    double* Ul = lds + M;
    const int32_t SL = ML ? HK_LSLOTS(BL, NCB) : 0, NL = ML ? NBK * NCB : 0;   // slots of a block, lists of the segment
    uint2* stage = reinterpret_cast<uint2*>(lds + 2 * M);
    int32_t* cw = reinterpret_cast<int32_t*>(stage + NBK * SL);
    int32_t* lb = cw + HK_PW * NBO;
    int32_t* lc = lb + NBO;              // [HK_PW][NL] counts, then places, of the lists
    int32_t* lg = lc + HK_PW * NL;       // [NBK] groups of the blocks
    __shared__ double anch[NBK + 1];             // time of the event before block j (j = NBK: the last event's)
    const int32_t s = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t a = s * HK_SEG;
    const int32_t b = a + HK_SEG < nev ? a + HK_SEG : nev;
    const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int32_t aw = a + wv * NBT * 64;
    int mks[NBT];
    double ts[NBT];
    float ws[NBT];
#pragma unroll
    for (int u = 0; u < NBT; ++u) {
        const int32_t i = aw + 64 * u + lane;
        const int32_t ic = i < b ? i : b - 1;
        mks[u] = clamp_mark(marks[c0 + ic], M);
        ts[u] = t[c0 + ic];
        ws[u] = wchunk[ic];
    }
    if (tid <= NBK) {
        const int32_t e = a + (tid << BL) < b ? a + (tid << BL) : b;   // the block's first event (past the end: b)
        anch[tid] = t[c0 + e > 0 ? c0 + e - 1 : 0];
    }
    for (int32_t k = tid; k < HK_PW * NBO; k += 64 * HK_PW) cw[k] = 0;
    int cbs[ML ? NBT : 1];               // the events' column blocks
    if constexpr (ML) {
        for (int32_t k = tid; k < HK_PW * NL; k += 64 * HK_PW) lc[k] = 0;
        for (int32_t k = tid; k < NBK * SL; k += 64 * HK_PW) stage[k] = make_uint2(0xffff0000u, 0u);
#pragma unroll
        for (int u = 0; u < NBT; ++u) cbs[u] = mks[u] / CW;
    }
    if (krow) {
        const double* cs = carry_seg + (int64_t)s * 2 * M;
        const double* gc = gcarry ? gcarry + (int64_t)(s / HK_SG) * 2 * M : nullptr;
        const double exg = gc ? seg_offdec[s] : 0.0;
        for (int32_t q = tid; q < M; q += 64 * HK_PW) {
            Kl[q] = gc ? __builtin_fma(exg, gc[q], cs[q]) : cs[q];
            Ul[q] = 0.0;
        }
    }
    __syncthreads();
    // the node blocks' starts for this segment (segment 0 stores the bases),
    // and each wave's events per node block
    if (wv == 0) {
        int32_t carry = 0;
        for (int32_t k0 = 0; k0 < NBO; k0 += 64) {
            const int32_t k = k0 + lane;
            const int32_t tot = k < NBO ? boff[(int64_t)k * (nseg + 1) + nseg] : 0;
            const int32_t off = k < NBO ? boff[(int64_t)k * (nseg + 1) + s] : 0;
            const int32_t incl = lane_incl_sum(tot, lane);
            if (k < NBO) {
                lb[k] = carry + incl - tot + off;
                if (s == 0) bbase[k] = carry + incl - tot;
            }
            carry += __shfl(incl, 63, 64);
        }
    }
    int32_t* run = cw + wv * NBO;
#pragma unroll
    for (int u = 0; u < NBT; ++u)
        if (aw + 64 * u + lane < b) {
            atomicAdd(&run[mks[u] >> bs], 1);
            if constexpr (ML) atomicAdd(&lc[wv * NL + ((wv * NBT + u) >> (BL - 6)) * NCB + cbs[u]], 1);
        }
    // factors of this wave's events
    const double bet = (double)beta[0];
    const double bl2 = bet * HK_LOG2E;   // decays as powers of 2
    float cf[NBT], bj[NBT];
#pragma unroll
    for (int u = 0; u < NBT; ++u) {
        const int jb = (wv * NBT + u) >> (BL - 6);
        const double d = ts[u] - anch[jb];
        cf[u] = (float)(bet * (double)ws[u]) * exp2_f64arg(-d * bl2);
        bj[u] = exp2_f64arg(d * bl2);
    }
    __syncthreads();
    for (int32_t k = tid; k < NBO; k += 64 * HK_PW) {
        int32_t p = lb[k];
#pragma unroll
        for (int v = 0; v < HK_PW; ++v) {
            const int32_t x = cw[v * NBO + k];
            cw[v * NBO + k] = p;
            p += x;
        }
    }
    if (ML && krow && tid < NBK) {
        // a thread a block: its lists' first groups, the waves' places in them
        int32_t g = 0;
        const int64_t blk = ((int64_t)a >> BL) + tid;
        const bool live = a + (tid << BL) < b;
        for (int32_t q = 0; q < NCB; ++q) {
            int32_t p = tid * SL + 64 * g;
            const int32_t p0 = p;
            for (int v = 0; v < HK_PW; ++v) {
                const int32_t x = lc[v * NL + tid * NCB + q];
                lc[v * NL + tid * NCB + q] = p;
                p += x;
            }
            if (live) plist[blk * (NCB + 1) + q] = g;
            g += (p - p0 + 63) >> 6;
        }
        if (live) plist[blk * (NCB + 1) + NCB] = g;
        lg[tid] = g;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NBT; ++u) {
        const int32_t base = aw + 64 * u;
        if (base >= b) break;
        const int32_t i = base + lane;
        const bool v = i < b;
        const int mk = mks[u];
        const int blk = mk >> bs;
        const uint64_t same = same_number(__ballot(v), blk, nbits);   // the lanes of this node block
        const int rank = __builtin_popcountll(same & lt);
        const int32_t before = run[blk];
        // 1 - e^{-x}: by subtraction when every event of the batch has x >= 0.5
        // (nothing cancels), else by expm1
        const double xT = bet * (T - ts[u]);
        const double em1 = __ballot(v && xT < 0.5) == 0 ? 1.0 - exp_f64(-xT) : -expm1(-xT);
        if (v) {
            const int32_t pos = before + rank;
            bo_e[pos] = em1;
            bo_key[pos] = ((uint32_t)i << bs) | (uint32_t)(mk & ((1 << bs) - 1));
            bo_cw[pos] = make_float2(cf[u], ws[u]);
        }
        uint64_t csame = 0;
        int32_t* lrun = nullptr;
        int32_t cat = 0;
        if constexpr (ML) {
            csame = same_number(__ballot(v), cbs[u], cbits);
            lrun = lc + wv * NL + ((wv * NBT + u) >> (BL - 6)) * NCB + cbs[u];
            cat = *lrun;
            if (v && krow)
                stage[cat + __builtin_popcountll(csame & lt)] =
                    make_uint2(((uint32_t)(i & ((1 << BL) - 1)) << 16) | (uint32_t)(8 * (mk - cbs[u] * CW)),
                               (uint32_t)__float_as_int(bj[u]));
        }
        lds_wait();   // every lane's read of the rank before the update
        if (v && (same & lt) == 0) run[blk] = before + __builtin_popcountll(same);
        if (ML && v && (csame & lt) == 0) *lrun = cat + __builtin_popcountll(csame);
        lds_wait();   // the update before the next batch's reads
        if (ML || !krow) continue;
        // pair record, at its place by bank (past the events: last)
        const int col = mk + M * (lane & (rep - 1));
        const int32_t pp = base + bank_place(v ? (col & 15) : 16, lt);
        prec[pp] = v ? make_uint2(((uint32_t)(i & ((1 << BL) - 1)) << 16) | (uint32_t)(8 * col),
                                  (uint32_t)__float_as_int(bj[u]))
                     : make_uint2(0xffff0000u, 0u);
    }
    if (!krow) return;
    if constexpr (ML) {
        __syncthreads();   // the stage is whole
        for (int j = 0; j < NBK; ++j) {
            uint2* o = prec + (((int64_t)a >> BL) + j) * SL;
            for (int32_t g = wv; g < lg[j]; g += HK_PW) {
                const uint2 x = stage[j * SL + 64 * g + lane];
                const bool v = (x.x >> 16) != 0xffffu;
                o[64 * g + bank_place(v ? (int)(x.x >> 3 & 15u) : 16, lt)] = x;
            }
        }
    }
    // groups past the last event of its block: records that precede nothing
#pragma unroll
    for (int u = 0; u < (ML ? 0 : NBT); ++u) {
        const int32_t base = aw + 64 * u;
        if (base >= b && (base >> BL) == ((b - 1) >> BL))
            prec[base + lane] = make_uint2(0xffff0000u | (uint32_t)(8 * (lane < M ? lane : 0)), 0u);
    }
    // the rows of K and U, block by block
    for (int j = 0; j < NBK && a + (j << BL) < b; ++j) {
        const int64_t blk = ((int64_t)a >> BL) + j;
        const double D = anch[j + 1] - anch[j];
        const double F = exp_f64(-bet * D);
        if (tid == 0) wide[blk] = !(bet * D <= HK_WIDE);
        RT* kr = krow + blk * Mp;
        for (int32_t q = tid; q < Mp; q += 64 * HK_PW) {
            const double k = q < M ? Kl[q] : 0.0;
            kr[krow_at<RT>(q)] = (RT)k;
            if (j + 1 < NBK && q < M) Kl[q] = k * F;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NBT; ++u) {
            if ((wv * NBT + u) >> (BL - 6) != j) continue;
            if (aw + 64 * u + lane < b) {
                if (j + 1 < NBK) atomicAdd(&Kl[mks[u]], exp_f64(-bet * (anch[j + 1] - ts[u])));
                atomicAdd(&Ul[mks[u]], (double)cf[u]);
            }
        }
        __syncthreads();
        RT* ur = urow + blk * Mp;
        for (int32_t q = tid; q < Mp; q += 64 * HK_PW) {
            ur[q] = q < M ? (RT)Ul[q] : (RT)0;
            if (q < M) Ul[q] = 0.0;
        }
    }
}

// Work item of a workgroup: consecutive items on one XCD (workgroups go round
// the 8 XCDs), so that the items of an event range share its L2.
__device__ __forceinline__ int32_t xcd_item(int32_t total) {
    const int32_t per = (total + 7) >> 3;
    const int32_t id = (int32_t)(blockIdx.x & 7u) * per + (int32_t)(blockIdx.x >> 3);
    return (int32_t)(blockIdx.x >> 3) < per && id < total ? id : -1;
}

// Workgroup (event range er of whole blocks, row block rb of 16 nodes, column
// block cb of CW nodes): the tile [16][CW] in float64 LDS.
//
// MC: several column blocks; the records come in a list per block of events and
// column block.
//
// Pair terms (waves HK_TGW and up): wave v a consecutive share of the range's
// blocks (fixed, so that the per-wave sums of dL/dmu and of the compensator
// add up in a fixed order).  Lanes are the records of a block; the own events
// of the row block (a stream of records in event order) are taken one after
// another, each adding c_i b_j at its row with one atomic per group of 64
// records up to its own.  The next block's records and the next 64 own records
// are in flight while a block is worked on.  Bound by the LDS float64 adds
// (about 10 cycles per 64 lanes and CU without bank conflicts, 24 at random
// columns: hence the permuted records).
//
// Product (waves 0 .. HK_TGW - 1): wave v the tiles of 16 x 16 columns of the
// column groups v, v + HK_TGW, ..; 16 x 16 x 4 MFMAs, float32 (the accumulators
// go to the tile every HK_FLUSH blocks; float32 sums over at most that many
// terms) or float64 (the layout's row64).  Lane l holds
// U[k + l / 16][row l mod 16], K[k + l / 16][column l mod 16]; result register
// r is row 4 (l / 16) + r (float32) or 4 r + l / 16 (float64), column l mod 16.
//
// Issue priority: the product waves last (their products fill the pair waves'
// gaps), a SIMD's pair waves in turn.  At equal priority the oldest wave goes
// first: the product ended at 72% and the pair waves at 82 to 100% of the
// launch (M = 1000, 2^20 events: 174 us; 158 now).
//
// PAIRS = false: the sums per node only.
#define HK_TW 16      // waves
#define HK_TGW 4      // of them on the product
#define HK_TPD 2      // steps of 4 blocks whose rows are in flight
#define HK_FLUSH 128
struct OwnRec {
    uint32_t key;
    float2 cw;
    double e;
};
template <int NG>
struct BlkRec {
    uint32_t key[NG];   // place in the block << 16 | 8 column
    float b[NG];
    int32_t wide;
};
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Raw buffer reads at a wave-uniform base: the lane's offset is a constant of
// the loop, so a load takes no vector instruction for its address; reads past
// the end return zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf(const void* p, int32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, bytes, 0x00020000);
}

// The product's part of the tile over blocks [kA, kB), the tile's nc columns
// that are nodes, this wave's GM column groups (a template parameter: with a branch around a load or a product the
// compiler's waits cover loads just issued).
template <int GM>
__device__ __forceinline__ void tile_product(const float* __restrict__ urow, const float* __restrict__ krow,
                                             int32_t Mp, int32_t r0, int32_t cb0, int32_t CW, int32_t nc, int32_t kA,
                                             int32_t kB, int wv, int lane, double* GP) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    f32x4 acc[GM][4] = {};
    f32x4 kv[HK_TPD][GM];
    float uv[HK_TPD];
    const int32_t vu = ((lane >> 4) * Mp + r0 + (lane & 15)) * 4;
    const int32_t vk = ((lane >> 4) * Mp + cb0 + wv * 64) * 4 + (lane & 15) * 16;
    auto fetch = [&](int32_t k, float& u, f32x4 (&x)[GM]) __attribute__((always_inline)) {
        // blocks past the range read as zero
        const int32_t left = uniform(kB - k < 0 ? 0 : kB - k < 4 ? kB - k : 4);
        const int64_t o = (int64_t)uniform(left > 0 ? k : kA) * Mp;
        const __amdgpu_buffer_rsrc_t rU = buf(urow + o, left * Mp * 4), rK = buf(krow + o, left * Mp * 4);
        u = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rU, vu, 0, 0));
#pragma unroll
        for (int g = 0; g < GM; ++g)
            x[g] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rK, vk + g * (HK_TGW * 256), 0, 0));
    };
    auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < GM; ++g)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int32_t col = (wv + HK_TGW * g) * 64 + c * 16 + (lane & 15);
                if (col < nc) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) atomicAdd(&GP[(4 * (lane >> 4) + r) * CW + col], (double)acc[g][c][r]);
                }
                acc[g][c] = f32x4{};
            }
    };
    int nacc = 0;
#pragma unroll
    for (int p = 0; p < HK_TPD; ++p) fetch(kA + 4 * p, uv[p], kv[p]);
    for (int32_t k = kA; k < kB; k += 4 * HK_TPD) {
#pragma unroll
        for (int p = 0; p < HK_TPD; ++p) {
#pragma unroll
            for (int g = 0; g < GM; ++g)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[g][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(uv[p], kv[p][g][c], acc[g][c], 0, 0, 0);
            fetch(k + 4 * (HK_TPD + p), uv[p], kv[p]);
        }
        nacc += 4 * HK_TPD;
        if (nacc + 4 * HK_TPD > HK_FLUSH) {
            flush();
            nacc = 0;
        }
    }
    if (nacc) flush();
}

// the same in float64 (groups of 32 columns)
template <int GM>
__device__ __forceinline__ void tile_product(const double* __restrict__ urow, const double* __restrict__ krow,
                                             int32_t Mp, int32_t r0, int32_t cb0, int32_t CW, int32_t nc, int32_t kA,
                                             int32_t kB, int wv, int lane, double* GP) {
    typedef double f64x2 __attribute__((ext_vector_type(2)));
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    f64x4 acc[GM][2] = {};
    f64x2 kv[HK_TPD][GM];
    double uv[HK_TPD];
    const int32_t vu = ((lane >> 4) * Mp + r0 + (lane & 15)) * 8;
    const int32_t vk = ((lane >> 4) * Mp + cb0 + wv * 32) * 8 + (lane & 15) * 16;
    auto fetch = [&](int32_t k, double& u, f64x2 (&x)[GM]) __attribute__((always_inline)) {
        const int32_t left = uniform(kB - k < 0 ? 0 : kB - k < 4 ? kB - k : 4);
        const int64_t o = (int64_t)uniform(left > 0 ? k : kA) * Mp;
        const __amdgpu_buffer_rsrc_t rU = buf(urow + o, left * Mp * 8), rK = buf(krow + o, left * Mp * 8);
        u = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rU, vu, 0, 0));
#pragma unroll
        for (int g = 0; g < GM; ++g)
            x[g] = __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(rK, vk + g * (HK_TGW * 256), 0, 0));
    };
#pragma unroll
    for (int p = 0; p < HK_TPD; ++p) fetch(kA + 4 * p, uv[p], kv[p]);
    for (int32_t k = kA; k < kB; k += 4 * HK_TPD) {
#pragma unroll
        for (int p = 0; p < HK_TPD; ++p) {
#pragma unroll
            for (int g = 0; g < GM; ++g)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[g][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(uv[p], kv[p][g][c], acc[g][c], 0, 0, 0);
            fetch(k + 4 * (HK_TPD + p), uv[p], kv[p]);
        }
    }
#pragma unroll
    for (int g = 0; g < GM; ++g)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int32_t col = (wv + HK_TGW * g) * 32 + c * 16 + (lane & 15);
            if (col < nc) {
#pragma unroll
                for (int r = 0; r < 4; ++r) atomicAdd(&GP[(4 * r + (lane >> 4)) * CW + col], acc[g][c][r]);
            }
        }
}

template <int BL, typename RT, bool PAIRS, bool MC>
__global__ __launch_bounds__(64 * HK_TW) void dense_tiles(int64_t c0, int32_t nev, int32_t M, int32_t Mp, int32_t CW,
                                                          int32_t NCB, int32_t NBO, int32_t ER, int32_t nseg,
                                                          const double* __restrict__ t,
                                                          const float* __restrict__ beta,
                                                          const int32_t* __restrict__ bo_off,
                                                          const int32_t* __restrict__ bo_base,
                                                          const uint32_t* __restrict__ bo_key,
                                                          const float2* __restrict__ bo_cw,
                                                          const double* __restrict__ bo_e,
                                                          const uint2* __restrict__ prec,
                                                          const int32_t* __restrict__ wide,
                                                          const RT* __restrict__ urow, const RT* __restrict__ krow,
                                                          double* __restrict__ gpart, double* __restrict__ spart,
                                                          double* __restrict__ cpart, int first, int32_t rep,
                                                          const int32_t* __restrict__ plist) {
    static_assert(HK_CW64 <= 32 * HK_TGW * 3, "float64 rows: at most three column groups a wave");
    // groups of 64 records per block; MC: of a list, held at a time
    constexpr int NG = MC && BL > 8 ? 6 : 1 << (BL - 6);
    constexpr int NPW = HK_TW - HK_TGW;
    extern __shared__ double lds[];
    double* Sw = lds;               // [NPW][16] sums of w per wave and row
    double* Ew = Sw + NPW * 16;     // [NPW][16] sums of the compensator terms
    double* GP = Ew + NPW * 16;     // [16][CW]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t id = xcd_item(NBO * NCB * ER);
    if (id < 0) return;
    // wave-uniform (the divisions run on the vector unit)
    const int32_t er = uniform(id / (NBO * NCB));
    const int32_t rb = uniform((id % (NBO * NCB)) / NCB), cb = uniform(id % NCB);
    const int32_t cb0 = cb * CW;
    const int32_t nblk = (nev + (1 << BL) - 1) >> BL;
    const int32_t rA = uniform((int32_t)((int64_t)er * nblk / ER));
    const int32_t rB = uniform((int32_t)((int64_t)(er + 1) * nblk / ER));
    for (int x = tid; x < 2 * NPW * 16; x += 64 * HK_TW) Sw[x] = 0.0;
    if (PAIRS)
        for (int x = tid; x < 16 * CW; x += 64 * HK_TW) GP[x] = 0.0;
    __syncthreads();
    if (wv < HK_TGW) {
        if constexpr (PAIRS) {
            __builtin_amdgcn_s_setprio(0);
            // this wave's column groups of 64 (float32) or 32 (float64)
            constexpr int GC = 256 / sizeof(RT);
            const int nm = (((CW + GC - 1) / GC) - wv + HK_TGW - 1) / HK_TGW;
            auto product = [&](auto gm) {
                tile_product<decltype(gm)::value>(urow, krow, Mp, rb * 16, cb0, CW, M - cb0 < CW ? M - cb0 : CW, rA,
                                                  rB, wv, lane, GP);
            };
            if (rA >= rB || nm <= 0) {
            } else if (nm == 1) {
                product(std::integral_constant<int, 1>{});
            } else if (nm == 2) {
                product(std::integral_constant<int, 2>{});
            } else if (nm == 3 || sizeof(RT) == 8) {   // (float64: HK_CW64 columns at most)
                product(std::integral_constant<int, 3>{});
            } else {
                product(std::integral_constant<int, 4>{});
            }
        }
    } else {
        const double bet = (double)beta[0];
        const double bl2 = bet * HK_LOG2E;
        const int pw = wv - HK_TGW;
        int rot = pw >> 2;
        const int32_t* off = bo_off + (int64_t)rb * (nseg + 1);
        const int32_t ob = bo_base[rb];
        // this wave's blocks and own records
        const int32_t kA = uniform(rA + (int32_t)((int64_t)pw * (rB - rA) / NPW));
        const int32_t kB = uniform(rA + (int32_t)((int64_t)(pw + 1) * (rB - rA) / NPW));
        const int32_t O1 = ob + off[(int32_t)(((int64_t)kB + (1 << (10 - BL)) - 1) >> (10 - BL))];   // or later
        int32_t oL = ob + off[kA >> (10 - BL)];   // first record of the batch in hand
        auto own_load = [&](OwnRec& o, int32_t from) {
            const int32_t e = from + lane < O1 ? from + lane : O1 - 1;
            o.key = bo_key[e];
            o.cw = bo_cw[e];
            if (!MC || cb == 0) o.e = bo_e[e];
        };
        auto blk_of = [&](const OwnRec& o) { return (int32_t)(o.key >> (4 + BL)); };
        auto own_sums = [&](const OwnRec& o, int32_t from) {
            if ((!MC || cb == 0) && from + lane < O1 && blk_of(o) >= kA && blk_of(o) < kB) {
                const int row = (int)(o.key & 15u);
                atomicAdd(&Sw[pw * 16 + row], (double)o.cw.y);
                atomicAdd(&Ew[pw * 16 + row], o.e);
            }
        };
        if (kA < kB && oL < O1) {
            // the records of the segment's earlier blocks: another wave's
            for (; oL < O1; oL += 64) {
                const int32_t e = oL + lane < O1 ? oL + lane : O1 - 1;
                const uint64_t bef = __ballot(oL + lane < O1 && (int32_t)(bo_key[e] >> (4 + BL)) < kA);
                if (~bef) {
                    oL += __builtin_popcountll(bef);
                    break;
                }
            }
        }
        if (kA < kB && oL < O1) {
            // MC: the groups [x, y) of the block's list for this column block
            const __amdgpu_buffer_rsrc_t rP = buf(prec, MC ? 0 : nblk << (BL + 3)), rW = buf(wide, nblk * 4);
            const __amdgpu_buffer_rsrc_t rL = buf(plist, MC ? nblk * (NCB + 1) * 4 : 0);
            auto ext_load = [&](int32_t blk) {
                const int32_t bc = (blk < nblk ? blk : nblk - 1) * ((NCB + 1) * 4);
                int2 e = make_int2(0, 0);
                if constexpr (MC)
                    e = make_int2((int)__builtin_amdgcn_raw_buffer_load_b32(rL, 0, bc + cb * 4, 0),
                                  (int)__builtin_amdgcn_raw_buffer_load_b32(rL, 0, bc + cb * 4 + 4, 0));
                return e;
            };
            // (MC: the groups from g0 to g1 of the block; past g1 zero, not read)
            auto blk_load = [&](BlkRec<NG>& r, int32_t blk, int32_t g0, int32_t g1) {
                const int32_t bc = blk < nblk ? blk : nblk - 1;
                const __amdgpu_buffer_rsrc_t rB =
                    MC ? buf(prec + (int64_t)bc * HK_LSLOTS(BL, NCB) + g0 * 64, (g1 - g0) * 512) : rP;
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const u32x2 x = __builtin_bit_cast(
                        u32x2,
                        __builtin_amdgcn_raw_buffer_load_b64(rB, lane * 8 + g * 512, MC ? 0 : bc << (BL + 3), 0));
                    r.key[g] = x.x;
                    r.b[g] = __int_as_float((int)x.y);
                }
                r.wide = __builtin_amdgcn_raw_buffer_load_b32(rW, 0, bc * 4, 0);
            };
            OwnRec oc, on;
            own_load(oc, oL);
            own_load(on, oL + 64);
            BlkRec<NG> rc, rn;
            // the first block's groups, and the next block's extent (in flight)
            int32_t gx = 0, gy = 0;
            int2 en = make_int2(0, 0);
            if (PAIRS) {
                if constexpr (MC) {
                    const int2 e = ext_load(kA);
                    gx = uniform(e.x);
                    gy = uniform(e.y);
                }
                blk_load(rc, kA, gx, gy);
                en = ext_load(kA + 1);
            }
            own_sums(oc, oL);
            int k = 0;         // own records of oc done
            // per own record of the batch: its block, and (byte offset of its
            // row in the tile) << 10 | place in the block; the valid lanes
            int32_t ob_;
            int pack;
            uint64_t todo;
            auto own_prep = [&]() {
                ob_ = blk_of(oc);
                pack = ((int)(oc.key & 15u) * (8 * CW)) << 10 | (int)((oc.key >> 4) & ((1u << BL) - 1u));
                todo = __ballot(oL + lane < O1);
            };
            own_prep();
            char* tile = reinterpret_cast<char*>(GP);
            for (int32_t blk = kA; PAIRS ? blk < kB : oL + 64 < O1; ++blk) {
                if (!PAIRS) {
                    oc = on;
                    oL += 64;
                    own_load(on, oL + 64);
                    own_sums(oc, oL);
                    continue;
                }
                // a SIMD's three pair waves take turns at the front
                rot = rot == 2 ? 0 : rot + 1;
                if (rot == 0)
                    __builtin_amdgcn_s_setprio(1);
                else if (rot == 1)
                    __builtin_amdgcn_s_setprio(2);
                else
                    __builtin_amdgcn_s_setprio(3);
                const int32_t nx = uniform(en.x), ny = uniform(en.y);
                blk_load(rn, blk + 1, nx, ny);
                en = ext_load(blk + 2);
                const bool w = __builtin_amdgcn_readfirstlane(rc.wide) != 0;
                int pl[NG];
                double bj[NG];
                uint32_t col[NG];   // byte offset of the column in the tile's row
                auto unpack = [&]() {
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
                        pl[g] = !MC || gx + g < gy ? (int)(rc.key[g] >> 16) : 0xffff;
                        col[g] = rc.key[g] & 0xffffu;
                        bj[g] = (double)rc.b[g];
                    }
                };
                unpack();
                const int32_t oL0 = oL;   // the block's first own record
                const int k0 = k;
                for (bool again = false;; again = true) {
                    for (;;) {
                        const uint64_t in = __ballot(ob_ == blk) & todo;
                        const int kn = k + __builtin_popcountll(in);
                        if (kn > k && !w) {
                            for (int x = k; x < kn; ++x) {
                                const int pk = rl_i(pack, x);
                                const double c = (double)rl_f(oc.cw.x, x);
                                char* row = tile + (pk >> 10);
                                const int pi = pk & 1023;
                                if constexpr (MC) {
                                    // a list's groups in event order: up to the
                                    // first without a record before the event
#pragma unroll
                                    for (int g = 0; g < NG; ++g) {
                                        const bool on = pl[g] < pi;
                                        if (__ballot(on) == 0) break;
                                        if (on) atomicAdd(reinterpret_cast<double*>(row + col[g]), c * bj[g]);
                                    }
                                    continue;
                                }
                                // the records before the event, group by group up
                                // to its own; the others' lanes add a zero (their
                                // high word cleared: at most a denormal), which
                                // costs one select instead of an exec mask and a
                                // branch
                                auto add = [&](int g) __attribute__((always_inline)) {
                                    const double v = c * bj[g];
                                    const int hi = pl[g] < pi ? __double2hiint(v) : 0;
                                    atomicAdd(reinterpret_cast<double*>(row + col[g]),
                                              __hiloint2double(hi, __double2loint(v)));
                                };
                                add(0);
                                if (NG > 1 && pi >= 64) {
                                    add(NG > 1 ? 1 : 0);
                                    if (NG > 2 && pi >= 128) {
                                        add(NG > 2 ? 2 : 0);
                                        if (pi >= 192) add(NG > 2 ? 3 : 0);
                                    }
                                }
                            }
                        } else if (kn > k) {
                            // wide block (the anchored factors could leave float32
                            // range): exact decays per pair
                            const int64_t b0 = c0 + ((int64_t)blk << BL);
                            double tr[NG];
#pragma unroll
                            for (int g = 0; g < NG; ++g) tr[g] = t[pl[g] < (1 << BL) ? b0 + pl[g] : b0];
                            const double town = t[c0 + (int32_t)(oc.key >> 4)];
                            const double cwd = bet * (double)oc.cw.y;
                            for (int x = k; x < kn; ++x) {
                                const int pk = rl_i(pack, x);
                                char* row = tile + (pk >> 10);
                                const int pi = pk & 1023;
                                const double tk = rl_d(town, x), ck = rl_d(cwd, x);
#pragma unroll
                                for (int g = 0; g < NG; ++g)
                                    if (pl[g] < pi)
                                        atomicAdd(reinterpret_cast<double*>(row + col[g]),
                                                  ck * (double)exp2_f64arg((tr[g] - tk) * bl2));
                            }
                        }
                        k = kn;
                        if (k < 64 || oL + 64 >= O1) break;
                        // oc used up: continue in on
                        oc = on;
                        oL += 64;
                        k = 0;
                        own_load(on, oL + 64);
                        if (!again) own_sums(oc, oL);
                        own_prep();
                    }
                    if (!MC || gx + NG >= gy) break;
                    // a list of more groups than are held: the next ones, and the
                    // block's own records again
                    gx += NG;
                    blk_load(rc, blk, gx, gy);
                    unpack();
                    if (oL != oL0) {
                        oL = oL0;
                        own_load(oc, oL);
                        own_load(on, oL + 64);
                        own_prep();
                    }
                    k = k0;
                }
                rc = rn;
                gx = nx;
                gy = ny;
            }
        }
    }
    __syncthreads();
    if (!MC || cb == 0)
        for (int x = tid; x < 16; x += 64 * HK_TW) {
            const int32_t row = rb * 16 + x;
            if (row >= M) continue;
            double sv = 0.0, ev = 0.0;
            for (int v = 0; v < NPW; ++v) {
                sv += Sw[v * 16 + x];
                ev += Ew[v * 16 + x];
            }
            const int64_t o = (int64_t)er * M + row;
            spart[o] = first ? sv : spart[o] + sv;
            cpart[o] = first ? ev : cpart[o] + ev;
        }
    if (!PAIRS) return;
    double* gp = gpart + (int64_t)er * M * M;
    for (int x = tid; x < 16 * CW; x += 64 * HK_TW) {
        const int32_t row = rb * 16 + x / CW, colm = cb0 + x % CW;
        if (row < M && colm < M) {
            const int64_t o = (int64_t)row * M + colm;
            double v = GP[x];
            for (int r = 1; r < rep; ++r) v += GP[x + r * M];   // the node's other columns
            gp[o] = first ? v : gp[o] + v;
        }
    }
}

// ------------------------------------------------------------------ host
static size_t prep_lds(const LargeArgs& A) {
    const size_t nbk = HK_SEG >> A.BL;
    const size_t lists = A.NCB > 1 ? nbk * (HK_LSLOTS(A.BL, A.NCB) * sizeof(uint2) +
                                            (HK_PW * A.NCB + 1) * sizeof(int32_t)) : 0;
    return (size_t)2 * A.M * sizeof(double) + lists + (size_t)(HK_PW + 1) * A.NBO * sizeof(int32_t);
}
static size_t tiles_lds(const LargeArgs& A, bool pairs) {
    return (2 * (HK_TW - HK_TGW) * 16 + (pairs ? (size_t)16 * A.CW : 0)) * sizeof(double);
}

// f(block length, several column blocks, row type) for the layout's choice
template <typename F>
static hawkes_status by_layout(const LargeArgs& A, F&& f) {
    auto go = [&](auto bl, auto mc) { return A.row64 ? f(bl, mc, (double*)nullptr) : f(bl, mc, (float*)nullptr); };
    if (A.NCB > 1) {
        if (A.BL == 10) return go(std::integral_constant<int, 10>{}, std::true_type{});
        if (A.BL == 9) return go(std::integral_constant<int, 9>{}, std::true_type{});
        return go(std::integral_constant<int, 8>{}, std::true_type{});
    }
    if (A.BL == 8) return go(std::integral_constant<int, 8>{}, std::false_type{});
    if (A.BL == 7) return go(std::integral_constant<int, 7>{}, std::false_type{});
    return go(std::integral_constant<int, 6>{}, std::false_type{});
}

hawkes_status dense_allow_lds(const LargeArgs& A) {
    return by_layout(A, [&](auto bl, auto mc, auto* rp) {
        constexpr int BL = decltype(bl)::value;
        constexpr bool MC = decltype(mc)::value;
        using RT = std::remove_pointer_t<decltype(rp)>;
        if (allow_lds((const void*)dense_prep<BL, RT, MC>, prep_lds(A)) != HAWKES_OK) return HAWKES_EUNSUPPORTED;
        if (A.support) return HAWKES_OK;
        return allow_lds((const void*)dense_tiles<BL, RT, true, MC>, tiles_lds(A, true));
    });
}

void large_dense_launch(LargeArgs& A, int64_t c0, int64_t c1, int32_t nseg, hipStream_t st, bool first,
                        bool sums_only) {
    const int32_t nev = (int32_t)(c1 - c0);
    int nbits = 0, cbits = 0;
    while ((1 << nbits) < A.NBO) ++nbits;
    while ((1 << cbits) < A.NCB) ++cbits;
    by_layout(A, [&](auto bl, auto mc, auto* rp) {
        constexpr int BL = decltype(bl)::value;
        constexpr bool MC = decltype(mc)::value;
        using RT = std::remove_pointer_t<decltype(rp)>;
        RT *ur = (RT*)A.urow, *kr = (RT*)A.krow;
        {
            TimedScope tk(7, st);
            hipLaunchKernelGGL((dense_prep<BL, RT, MC>), dim3(nseg), dim3(64 * HK_PW), prep_lds(A), st, c0, nev, A.M,
                               A.Mp, A.NBO, nbits, 4, A.T, A.t, A.marks, A.wchunk, A.beta, A.carry_seg,
                               A.carry_prefix ? A.gcarry : (const double*)nullptr, A.seg_offdec, nseg, A.bo_off,
                               A.bo_base, A.bo_key, A.bo_cw, A.bo_e, A.prec, A.wide, ur,
                               sums_only ? (RT*)nullptr : kr, A.rep, A.CW, A.NCB, cbits, A.plist);
        }
        TimedScope ts(0, st);
        auto tiles = [&](auto* kern, bool pairs, int32_t ncb) {
            const int32_t items = A.NBO * ncb * A.ER;
            hipLaunchKernelGGL(kern, dim3((unsigned)(((items + 7) / 8) * 8)), dim3(64 * HK_TW), tiles_lds(A, pairs),
                               st, c0, nev, A.M, A.Mp, A.CW, ncb, A.NBO, A.ER, nseg, A.t, A.beta, A.bo_off,
                               A.bo_base, A.bo_key, A.bo_cw, A.bo_e, A.prec, A.wide, ur, kr, A.gpart, A.spart,
                               A.cpart_, first ? 1 : 0, A.rep, A.plist);
        };
        if (sums_only)
            tiles(dense_tiles<BL, RT, false, false>, false, 1);
        else
            tiles(dense_tiles<BL, RT, true, MC>, true, A.NCB);
        return HAWKES_OK;
    });
}

}  // namespace hk
