// Large-M engine: one sequence, M > 8 nodes, decay shared by all targets.
//
// The sequence is evaluated in chunks of CH events (constant memory: only
// M-vector carries cross a chunk boundary, as in the batched procedure of
// Algorithm 2).  Within a chunk, segments of HK_SEG events are the scan
// elements.  The state is the source-indexed pair of the paper's gradient
// recurrence (eq. 11) and its time-weighted companion:
//   K_q(t) = sum_{j: t_j<t, m_j=q} e^{-beta (t - t_j)}
//   J_q(t) = sum_{j: t_j<t, m_j=q} (t - t_j) e^{-beta (t - t_j)}
// A run of events maps the state at its start to the state at its end by
//   K -> e^{-beta D} K + K_run,   J -> e^{-beta D} (J + D K) + J_run
// (the (s I, v) maps of "Methods", with a shear for J); composing these is
// the associative operator of the scan.
//
// Per chunk:
//   agg      one wave per segment folds its events into (K_run, J_run)
//   scan     one thread per node chains the segment maps -> carry-in per segment
//   forward  a workgroup of four waves per segment (two with many nodes) replays
//            its events 64 at a time, one per lane; a wave takes a share of each
//            event's row of alpha, the first adds the partial sums and forms the
//            intensity, another the compensator terms, another updates the
//            records.  Each node keeps a record (K_q, J_q) in LDS, anchored at
//            the segment's start (with a time of its own where the anchored
//            exponents could overflow); lambda_i needs only the nonzeros of
//            alpha's row m_i (R = alpha_{m_i,:} . K, eq. 3), read from a CSR copy
//            of alpha, plus the same-batch events found through a per-node lane
//            mask.  It writes lambda_i / per-segment float64 partials and, for
//            the gradient, per-event coefficients for the dense kernel.
//   bucket   the starts of the partition of the chunk's events by blocks of 16
//            nodes (hk_bucket.hip)
//   dense    dense dL/dalpha (first term of eq. 9, hk_dense.hip): per block of
//            events the state's rows and the events' records, then tiles of 16
//            rows per event range, pair terms and matrix product side by side
#include "hk_device.h"
#include "hk_large.h"
#include <stdlib.h>
#include <mutex>

namespace hk {

// ------------------------------------------------------------------ setup
// alpha as the passes read it, and the call's cleared state, in two launches
// (they were one kernel per array, 8 to 12 launches of about 5 us each):
//   large_setup   workgroups of 16 waves by role: column sums of alpha (64
//                 columns; wave r sums rows r, r + 16, .., coalesced over the
//                 columns, then a fixed-order sum), nonzeros per row (16 rows,
//                 a wave a row), cleared arrays
//   large_index   a wave a row: the row's start (the sum of the counts before
//                 it), its nonzeros in column order, and its node record
//                 (csr begin, csr end, mu, colsum): one 16-byte load per event;
//                 gsup (or null): the sums in the order of the nonzeros, cleared
//                 in each of the ncopy copies
// With trans the rows are the columns of alpha (compressed-column form).
// blockIdx.y: the decay kernel.
__device__ __forceinline__ float alpha_at(const float* __restrict__ alpha, int32_t M, int32_t r, int32_t c,
                                          int trans) {
    return trans ? alpha[(int64_t)c * M + r] : alpha[(int64_t)r * M + c];
}

__global__ __launch_bounds__(1024) void large_setup(int32_t M, const float* __restrict__ alpha, int trans, int32_t NC,
                                                    int32_t NR, float* __restrict__ colsum,
                                                    int32_t* __restrict__ rcnt, ZeroList Z) {
    __shared__ double part[16][64];
    const int lane = threadIdx.x & 63, r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t k = blockIdx.y;
    alpha += (int64_t)k * M * M;
    int32_t blk = blockIdx.x;
    if (blk < NC) {
        const int32_t q = blk * 64 + lane;
        double c = 0.0;
        if (q < M) {
#pragma unroll 8
            for (int32_t p = r; p < M; p += 16) c += (double)alpha[(int64_t)p * M + q];
        }
        part[r][lane] = c;
        __syncthreads();
        if (r == 0 && q < M) {
            double v = 0.0;
            for (int i = 0; i < 16; ++i) v += part[i][lane];
            colsum[(int64_t)k * M + q] = (float)v;
        }
        return;
    }
    blk -= NC;
    if (blk < NR) {
        const int32_t p = blk * 16 + r;
        if (p >= M) return;
        int32_t cnt = 0;
#pragma unroll 4
        for (int32_t q = lane; q < M; q += 64) cnt += alpha_at(alpha, M, p, q, trans) != 0.0f;
        for (int off = 32; off > 0; off >>= 1) cnt += __shfl_down(cnt, off, 64);
        if (lane == 0) rcnt[(int64_t)k * M + p] = cnt;
        return;
    }
    if (k > 0) return;
    blk -= NR;
    const int32_t nz = (int32_t)gridDim.x - NC - NR;
    for (int z = 0; z < HK_NZERO; ++z)
        for (int64_t i = blk * 1024ll + threadIdx.x; i < Z.n[z]; i += nz * 1024ll) Z.p[z][i] = 0.0;
}

__global__ __launch_bounds__(1024) void large_index(int32_t M, const float* __restrict__ alpha, int trans,
                                                    const int32_t* __restrict__ rcnt, int32_t* __restrict__ ptr,
                                                    int2* __restrict__ cv, int64_t cvs, const float* __restrict__ mu,
                                                    const float* __restrict__ colsum, int4* __restrict__ node_info,
                                                    const float* __restrict__ beta, float* __restrict__ csc_b,
                                                    double* __restrict__ gsup, int32_t ncopy) {
    const int lane = threadIdx.x & 63, r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t k = blockIdx.y, p = blockIdx.x * 16 + r;
    if (p >= M) return;
    alpha += (int64_t)k * M * M;
    rcnt += (int64_t)k * M;
    ptr += (int64_t)k * (M + 1);
    cv += k * cvs;
    int32_t o = 0;
#pragma unroll 4
    for (int32_t i = lane; i < p; i += 64) o += rcnt[i];
    for (int off = 32; off > 0; off >>= 1) o += __shfl_xor(o, off, 64);
    const int32_t e = o + rcnt[p];
    if (lane == 0) {
        ptr[p] = o;
        if (p == M - 1) ptr[M] = e;
        if (node_info)
            node_info[(int64_t)k * M + p] =
                make_int4(o, e, __float_as_int(mu[p]), __float_as_int(colsum[(int64_t)k * M + p]));
    }
    for (int32_t q0 = 0; q0 < M; q0 += 64) {
        const int32_t q = q0 + lane;
        const float a = q < M ? alpha_at(alpha, M, p, q, trans) : 0.0f;
        const uint64_t nz = __ballot(a != 0.0f);
        if (a != 0.0f) {
            const int32_t i = o + __builtin_popcountll(nz & (lane ? (~0ull >> (64 - lane)) : 0ull));
            cv[i] = make_int2(q, __float_as_int(a));
            if (csc_b) csc_b[i] = beta[q];
            if (gsup)
                for (int32_t c = 0; c < ncopy; ++c) gsup[(int64_t)c * M * M + i] = 0.0;
        }
        o += __builtin_popcountll(nz);
    }
}

void large_setup_launch(const LargeArgs& A, int trans, bool colsums, bool index, const ZeroList& Z, hipStream_t st) {
    const int32_t NC = colsums ? (A.M + 63) / 64 : 0, NR = index ? (A.M + 15) / 16 : 0;
    int64_t total = 0;
    for (int z = 0; z < HK_NZERO; ++z) total += Z.n[z];
    const int64_t nz = total < 1024 * 1024 ? (total + 4095) / 4096 : 256;
    hipLaunchKernelGGL(large_setup, dim3((unsigned)(NC + NR + nz), (unsigned)A.K), dim3(1024), 0, st, A.M, A.alpha,
                       trans, NC, NR, A.colsum, A.rcnt, Z);
}

void large_index_launch(const LargeArgs& A, int trans, int32_t* ptr, int2* cv, int4* node_info, float* csc_b,
                        hipStream_t st, double* gsup, int32_t ncopy) {
    hipLaunchKernelGGL(large_index, dim3((unsigned)((A.M + 15) / 16), (unsigned)A.K), dim3(1024), 0, st, A.M, A.alpha,
                       trans, A.rcnt, ptr, cv, cv_stride((int64_t)A.M * A.M), A.mu, A.colsum, node_info, A.beta,
                       csc_b, gsup, ncopy);
}

// ------------------------------------------------------------------ agg
// one wave per segment; LDS: aggK[M], aggJ[M] (float64)
__global__ __launch_bounds__(64) void large_seg_agg(int64_t c0, int64_t c1, int32_t M, const double* __restrict__ t,
                                                    const int32_t* __restrict__ marks, const float* __restrict__ beta,
                                                    double* __restrict__ agg, double* __restrict__ seg_span,
                                                    double* __restrict__ seg_dec) {
    extern __shared__ double lds[];
    double* aK = lds;
    double* aJ = lds + M;
    const int32_t s = blockIdx.x;
    const int64_t a = c0 + (int64_t)s * HK_SEG;
    const int64_t b = a + HK_SEG < c1 ? a + HK_SEG : c1;
    const int lane = threadIdx.x;
    for (int32_t q = lane; q < M; q += 64) { aK[q] = 0.0; aJ[q] = 0.0; }
    __syncthreads();
    const double bet = (double)beta[0];
    const double te = t[b - 1];
    // the segment's times and marks, all loads issued up front (past the
    // end: a valid index, not added)
    constexpr int NBT = HK_SEG / 64;
    double ts[NBT];
    int mks[NBT];
#pragma unroll
    for (int u = 0; u < NBT; ++u) {
        const int64_t i = a + 64 * u + lane;
        const int64_t ic = i < b ? i : b - 1;
        ts[u] = t[ic];
        mks[u] = marks[ic];
    }
#pragma unroll
    for (int u = 0; u < NBT; ++u) {
        if (a + 64 * u + lane < b) {
            const double d = te - ts[u];
            const double e = exp_f64(-bet * d);
            const int mi = clamp_mark(mks[u], M);
            atomicAdd(&aK[mi], e);
            atomicAdd(&aJ[mi], d * e);
        }
    }
    __syncthreads();
    double* o = agg + (int64_t)s * 2 * M;
    for (int32_t q = lane; q < M; q += 64) { o[q] = aK[q]; o[M + q] = aJ[q]; }
    if (lane == 0) {
        // span and decay from the event before the segment to its last event
        const double tr = a > 0 ? t[a - 1] : t[a];
        seg_span[s] = te - tr;
        seg_dec[s] = exp(-bet * (te - tr));
    }
}

// ------------------------------------------------------------------ scan
// Segment maps are chained in three parallel steps (groups of HK_SG segments):
//   1 thread per (group, node): exclusive prefix inside the group, group map
//   2 thread per node: chain the group maps from the chunk carry
//   3 thread per (segment, node): carry_seg[s] = group carry moved to the
//     segment start, plus the in-group prefix
// carry_seg[s] is the state just after the event preceding segment s.

// beta_pt: per-target decays (R-form state) or nullptr (one shared decay,
// seg_dec / gdec precomputed)
// The threads also write the group's gspan/gdec and every segment's
// seg_off/seg_offdec: the time from the event before the group to the event
// before the segment, and its decay (shared decay beta[0]).
__global__ __launch_bounds__(256) void large_scan_local(int32_t nseg, int32_t M, const double* __restrict__ agg,
                                 const double* __restrict__ seg_dec, const double* __restrict__ seg_span,
                                 double* __restrict__ carry_seg, double* __restrict__ gagg,
                                 const float* __restrict__ beta_pt, const float* __restrict__ beta,
                                 double* __restrict__ gspan, double* __restrict__ gdec,
                                 double* __restrict__ seg_off, double* __restrict__ seg_offdec) {
    const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int32_t ngr = (nseg + HK_SG - 1) / HK_SG;
    if (gid >= (int64_t)ngr * M) return;
    const int32_t g = (int32_t)(gid / M), q = (int32_t)(gid % M);
    const int32_t s0 = g * HK_SG, s1 = s0 + HK_SG < nseg ? s0 + HK_SG : nseg;
    // offset u of the group (u = 0 .. s1 - s0, the last one the group's
    // span) is summed by the threads q = u, u + M, ..: each sums the spans in
    // the same order as one serial pass would, so the values do not depend on
    // M, and the group's exps run side by side instead of one after another
    if (q <= s1 - s0) {
        // the group's spans, loaded together (not one dependent load per
        // term of the sum)
        double sp[HK_SG];
#pragma unroll
        for (int v = 0; v < HK_SG; ++v) sp[v] = seg_span[s0 + v < s1 ? s0 + v : s1 - 1];
    for (int32_t u = q; u <= s1 - s0; u += M) {
        const double b0 = (double)beta[0];
        double D = 0.0;
#pragma unroll
        for (int v = 0; v < HK_SG; ++v)
            if (v < u) D += sp[v];
        const double e = exp(-b0 * D);
        if (u < s1 - s0) {
            seg_off[s0 + u] = D;
            seg_offdec[s0 + u] = e;
        } else {
            gspan[g] = D;
            gdec[g] = e;
        }
    }
    }
    double K = 0.0, J = 0.0;
    const double bq = beta_pt ? (double)beta_pt[q] : 0.0;
    // the group's segment maps of node q, spans and decays, 16 segments at a
    // time: their loads and exponentials before the chain (two multiply-adds
    // a segment).  With the spans and decays read inside the chain it was 32
    // dependent loads (us a launch, M = 251: 12, 6 now; M = 1000: 13, 8).
    constexpr int PF = 16;
#pragma unroll
    for (int h = 0; h < HK_SG; h += PF) {
        double rk[PF], rj[PF], D[PF], ex[PF];
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int32_t s = s0 + h + u < s1 ? s0 + h + u : s1 - 1;
            rk[u] = agg[(int64_t)s * 2 * M + q];
            rj[u] = agg[(int64_t)s * 2 * M + M + q];
            D[u] = seg_span[s];
            ex[u] = beta_pt ? 0.0 : seg_dec[s];
        }
        if (beta_pt) {
#pragma unroll
            for (int u = 0; u < PF; ++u) ex[u] = exp(-bq * D[u]);
        }
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int32_t s = s0 + h + u;
            if (s < s1) {
                double* o = carry_seg + (int64_t)s * 2 * M;
                o[q] = K;
                o[M + q] = J;
                const double k0 = K;
                K = __builtin_fma(ex[u], k0, rk[u]);
                J = __builtin_fma(ex[u], __builtin_fma(D[u], k0, J), rj[u]);
            }
        }
    }
    gagg[(int64_t)g * 2 * M + q] = K;
    gagg[(int64_t)g * 2 * M + M + q] = J;
}

__global__ __launch_bounds__(256) void large_scan_groups(int32_t nseg, int32_t M, const double* __restrict__ gagg,
                                  const double* __restrict__ gspan, const double* __restrict__ gdec,
                                  double* __restrict__ gcarry, double* __restrict__ carry,
                                  const float* __restrict__ beta_pt) {
    const int32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= M) return;
    const int32_t ngr = (nseg + HK_SG - 1) / HK_SG;
    double K = carry[q], J = carry[M + q];
    const double bq = beta_pt ? (double)beta_pt[q] : 0.0;
    // 16 group maps of node q at a time, their loads and decays up front
    constexpr int PF = 16;
    for (int32_t g0 = 0; g0 < ngr; g0 += PF) {
        double gk[PF], gj[PF], D[PF], ex[PF];
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int32_t g = g0 + u < ngr ? g0 + u : ngr - 1;
            gk[u] = gagg[(int64_t)g * 2 * M + q];
            gj[u] = gagg[(int64_t)g * 2 * M + M + q];
            D[u] = gspan[g];
            ex[u] = beta_pt ? 0.0 : gdec[g];
        }
        if (beta_pt) {
#pragma unroll
            for (int u = 0; u < PF; ++u) ex[u] = exp(-bq * D[u]);
        }
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int32_t g = g0 + u;
            if (g < ngr) {
                gcarry[(int64_t)g * 2 * M + q] = K;
                gcarry[(int64_t)g * 2 * M + M + q] = J;
                const double k0 = K;
                K = __builtin_fma(ex[u], k0, gk[u]);
                J = __builtin_fma(ex[u], __builtin_fma(D[u], k0, J), gj[u]);
            }
        }
    }
    carry[q] = K;
    carry[M + q] = J;
}

__global__ void large_scan_apply(int32_t nseg, int32_t M, const double* __restrict__ seg_off,
                                 const double* __restrict__ seg_offdec, const double* __restrict__ gcarry,
                                 double* __restrict__ carry_seg, const float* __restrict__ beta_pt) {
    const int64_t gid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (gid >= (int64_t)nseg * M) return;
    const int32_t s = (int32_t)(gid / M), q = (int32_t)(gid % M);
    const int32_t g = s / HK_SG;
    const double D = seg_off[s];
    const double ex = beta_pt ? exp(-(double)beta_pt[q] * D) : seg_offdec[s];
    const double Kc = gcarry[(int64_t)g * 2 * M + q], Jc = gcarry[(int64_t)g * 2 * M + M + q];
    double* o = carry_seg + (int64_t)s * 2 * M;
    const double Kl = o[q], Jl = o[M + q];
    o[q] = __builtin_fma(ex, Kc, Kl);
    o[M + q] = __builtin_fma(ex, __builtin_fma(D, Kc, Jc), Jl);
}

// ------------------------------------------------------------------ forward
// Four waves per segment, in the 128 registers that let four of them share a
// SIMD (a chunk of 2^20 events has 1024 segments: with two waves each, and 190
// registers, two were on a SIMD and the pass waited more than half its time).
// Us a launch, two / four waves: M = 1000, 1e6 events, gradient 57 / 51,
// log-likelihood 51 / 43; M = 251, 3e5 events 52 / 40; M = 100, 1e6 events,
// intensities 56 / 47.  Two waves where four waves' sums and the records pass
// the LDS (M > HK_FW4_MAX_M).
#define HK_FW4_MAX_M 6400
// nonzeros of an event's row of alpha loaded one batch ahead (more of them
// with four waves cost registers: 24 spilled with 16)
constexpr int fwd_ahead(int nw) { return nw == 4 ? 8 : 16; }
// RM (several decay kernels): the pass runs once per kernel and writes, per
// event, R = alpha_{m_i,:} . K(t_i) to rk and (GRAD) D = alpha_{m_i,:} . J(t_i)
// to dk instead of forming lambda; large_combine then sums the kernels.
// SUPP (with GRAD): also adds beta w_i K_q(t_i) to gsup[k] for every nonzero
// k = (m_i, q) of alpha's CSR (hardware float64 atomics): the first term of
// eq. 9 on alpha's support only.  Segment s adds into copy s & cmask (copies
// MM apart): consecutive workgroups go to different XCDs, so each copy sees
// mostly one XCD's atomics and a copy's addresses see a fraction of the
// contention.
// X (optional parts, each off when its pointer is null):
//   gcarry    carry_seg holds only the in-group prefixes of the scan
//             (large_scan without its apply pass): the state entering segment
//             s is formed here from its group's carry, seg_off and seg_offdec
//   bcnt      the chunk partition's counts, events per (node block of 2^bs
//             nodes, segment), written as bucket_count would
// 1 / x for a positive normal float64 x: the hardware reciprocal and two
// Newton steps (within about 1 ulp; an IEEE division takes twice the
// instructions)
__device__ __forceinline__ double recip(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

template <bool GRAD, bool INTENS, bool SUPP, int NW, bool RM = false>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 4 ? 4 : 1))) void large_forward(int64_t c0, int64_t c1, int32_t M, double T,
                                                    const double* __restrict__ t, const int32_t* __restrict__ marks,
                                                    const float* __restrict__ mu, const float* __restrict__ beta,
                                                    const int4* __restrict__ node_info,
                                                    const int2* __restrict__ csr_cv,
                                                    const double* __restrict__ carry_seg,
                                                    double* __restrict__ seg_part,
                                                    float* __restrict__ wchunk,
                                                    float* __restrict__ lambda_out,
                                                    double* __restrict__ gsup, int32_t cmask,
                                                    double* __restrict__ rk, double* __restrict__ dk,
                                                    FwdExtra X) {
    extern __shared__ double lds[];
    double2* rKJ = reinterpret_cast<double2*>(lds);       // [M] (K_q, J_q) at rtau (event included)
    uint64_t* rmask = (uint64_t*)(lds + 2 * M);           // [M] lanes of this batch with mark q
    __shared__ double tb[64], eb[64];
    __shared__ double Rs[(NW > 1 ? NW - 1 : 1) * 64], Ds[(NW > 1 ? NW - 1 : 1) * 64];   // other waves' partial sums
    const int32_t s = blockIdx.x;
    const int lane = threadIdx.x & 63;
    // NW waves share a segment's events; wave wv takes the aligned pairs of
    // nonzeros wv, wv + NW, ... of each event's row of alpha
    const int wv = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr int WE = NW == 4 ? 1 : NW - 1;
    static_assert(!SUPP || NW == 1, "the support-restricted sums are formed by one wave");
    static_assert(!(RM && (SUPP || INTENS)), "per-kernel sums only");
    const int64_t a = c0 + (int64_t)s * HK_SEG;
    const int64_t b = a + HK_SEG < c1 ? a + HK_SEG : c1;
    const double bet = (double)beta[0];
    const double tref = a > 0 ? t[a - 1] : t[a];
    // anchored records when the segment's span allows: with u = t - tref,
    // rKJ[q] = (S0_q, S1_q) with S0_q = sum_j e^{beta u_j}, S1_q = sum_j u_j e^{beta u_j}
    // over the node's events so far (the carry enters as S0 = K(tref),
    // S1 = -J(tref)); then K_q(t) = e^{-beta u} S0_q and
    // J_q(t) = e^{-beta u} (u S0_q - S1_q): one exponential per event instead
    // of one per nonzero of alpha's row, and records grow by plain additions.
    // Otherwise (beta u could overflow float64) each record keeps its own
    // time rtau[q] and is decayed on use.
    const bool anch = bet * (t[b - 1] - tref) <= 600.0;
    // [M] the lazy records' times, in the segment's slot of a global scratch
    // buffer (24 bytes of LDS per node instead of 32: M up to 6741)
    double* rtau = X.rtau + (int64_t)s * 2 * M;
    const double* cs = carry_seg + (int64_t)s * 2 * M;
    const double* gc = X.gcarry ? X.gcarry + (int64_t)(s / HK_SG) * 2 * M : nullptr;
    const double Dg = gc ? X.seg_off[s] : 0.0, exg = gc ? X.seg_offdec[s] : 0.0;
    for (int32_t q = threadIdx.x; q < M; q += 64 * NW) {
        double Kq = cs[q], Jq = cs[M + q];
        if (gc) {
            // the group's carry moved to the segment start, plus the prefix
            const double Kc = gc[q];
            Jq = __builtin_fma(exg, __builtin_fma(Dg, Kc, gc[M + q]), Jq);
            Kq = __builtin_fma(exg, Kc, Kq);
        }
        if (!anch) rtau[q] = tref;
        rKJ[q] = make_double2(Kq, anch ? -Jq : Jq);
        rmask[q] = 0ull;
    }
    // events per node block (partition counts): dynamic LDS after the
    // records, present when bcnt is given
    int32_t* lcnt = reinterpret_cast<int32_t*>(lds + 3 * M);
    if (X.bcnt)
        for (int32_t k = threadIdx.x; k < X.nbo; k += 64 * NW) lcnt[k] = 0;
    __syncthreads();
    double logsum = 0.0, comp = 0.0, Esum = 0.0, gb = 0.0;
    // software pipeline over batches of 64 events: times and marks are loaded
    // three batches ahead, node records two ahead and the first FW nonzeros
    // of each event's row of alpha one ahead (clamped indices keep every load
    // valid), so the gathers' latency hides behind a batch of work.  The row
    // is read in aligned pairs of entries (pair P holds entries 2P and 2P + 1,
    // one 16-byte load; the first and last pair may hold a neighbour row's
    // entry, which is skipped): these gathers hit a different cache line per
    // lane, so the number of load instructions, not bytes, sets their cost.
    constexpr int FW = fwd_ahead(NW);  // nonzeros loaded ahead per event
    constexpr int FP = FW / (2 * NW);  // pairs of them loaded by this wave
    static_assert(FP >= 1 && FP * 2 * NW == FW, "look-ahead must be whole pairs per wave");
    const int4* __restrict__ cv4 = reinterpret_cast<const int4*>(csr_cv);
    auto ld_tm = [&](int64_t base, double& tt, int& mm) {
        const int64_t j = base + lane;
        const int64_t jc = j < b ? j : b - 1;
        tt = t[jc];
        mm = clamp_mark(marks[jc], M);
    };
    // pairs past the row's last entry are replaced by its first pair (an
    // empty row reads pair nv.x / 2, inside the array's one spare pair)
    auto ld_row = [&](const int4& nv, int4 (&pr)[FP]) {
        const int32_t p0 = nv.x >> 1, pl = (nv.y - 1) >> 1;
#pragma unroll
        for (int j = 0; j < FP; ++j) {
            const int32_t P = p0 + NW * j + wv;
            pr[j] = cv4[P <= pl ? P : p0];
        }
    };
    double t0, t1, t2;
    int m0, m1, m2;
    ld_tm(a, t0, m0);
    ld_tm(a + 64, t1, m1);
    ld_tm(a + 128, t2, m2);
    int4 n0 = node_info[m0], n1 = node_info[m1];
    int4 pr0[FP];
    ld_row(n0, pr0);
    for (int64_t base = a; base < b; base += 64) {
        // the waves with the batch's serial work go first
        if (NW > 1 && (wv == 0 || wv == NW - 1)) __builtin_amdgcn_s_setprio(2);
        const int64_t i = base + lane;
        const bool valid = i < b;
        const double ti = valid ? t0 : 0.0;
        const int mi = valid ? m0 : 0;
        const int4 ni = n0;
        // loads for the batches ahead
        const int4 n2 = node_info[m2];
        int4 pr1[FP];
        ld_row(n1, pr1);
        const double ui = ti - tref;
        // after the sums: the first wave the logarithm and reciprocal, wave WE
        // the compensator terms, wave WC the records (one wave: all of it)
        constexpr int WC = NW - 1;
        double eti = 0.0;   // e^{beta u_i} (anchored records; the first wave)
        if (wv == 0) {
            eti = anch && valid ? exp_f64(bet * ui) : 0.0;
            tb[lane] = ti;
            eb[lane] = eti;
            if (valid) atomicOr((unsigned long long*)&rmask[mi], 1ull << lane);
            if (X.bcnt && valid) atomicAdd(&lcnt[mi >> X.bs], 1);
        }
        __syncthreads();
        double R = 0.0, Dd = 0.0, lam = 1.0, w = 0.0, em1 = 0.0;
        const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
        const int32_t k0 = ni.x, k1 = ni.y, p0 = k0 >> 1;
        double ks[SUPP ? 2 * FP : 1];   // the loaded pairs' sums, for gsup (NW = 1)
            // anchored sums of source q (records plus the batch's earlier
            // events of q): K_q(t_i) = e^{-beta u_i} s0
            auto sums_a = [&](int32_t q, double& s0, double& s1) {
                const double2 kj = rKJ[q];   // one LDS read for both
                s0 = kj.x;
                s1 = GRAD ? kj.y : 0.0;
                uint64_t bits = rmask[q] & below;
                while (bits) {
                    const int jj = __builtin_ctzll(bits);
                    bits &= bits - 1;
                    const double ej = eb[jj];
                    s0 += ej;
                    if (GRAD) s1 = __builtin_fma(tb[jj] - tref, ej, s1);
                }
            };
            // source q's record decayed to ti plus the batch's earlier events
            // of q: Kv = K_q(t_i), Jv = J_q(t_i)
            auto sums_w = [&](int32_t q, double& Kv, double& Jv) {
                const double d = ti - rtau[q];
                const double e = exp_f64(-bet * d);
                const double2 kj = rKJ[q];
                const double kq = kj.x;
                Kv = e * kq;
                Jv = GRAD ? e * __builtin_fma(d, kq, kj.y) : 0.0;
                uint64_t bits = rmask[q] & below;
                while (bits) {
                    const int jj = __builtin_ctzll(bits);
                    bits &= bits - 1;
                    const double dj = ti - tb[jj];
                    const double ej = exp_f64(-bet * dj);
                    Kv += ej;
                    if (GRAD) Jv = __builtin_fma(dj, ej, Jv);
                }
            };
            if (!valid) {
            } else if (anch) {
                // source q with weight av
                auto terma = [&](int32_t q, float av) -> double {
                    double s0, s1;
                    sums_a(q, s0, s1);
                    R = __builtin_fma((double)av, s0, R);
                    if (GRAD) Dd = __builtin_fma((double)av, __builtin_fma(ui, s0, -s1), Dd);
                    return s0;
                };
#pragma unroll
                for (int j = 0; j < FP; ++j) {
                    const int32_t kb = 2 * (p0 + NW * j + wv);
                    if (kb < k1) {
                        if (kb >= k0) {
                            const double v = terma(pr0[j].x, __int_as_float(pr0[j].y));
                            if (SUPP) ks[2 * j] = v;
                        }
                        if (kb + 1 < k1) {
                            const double v = terma(pr0[j].z, __int_as_float(pr0[j].w));
                            if (SUPP) ks[2 * j + 1] = v;
                        }
                    }
                }
                for (int32_t kb = 2 * (p0 + NW * FP + wv); kb < k1; kb += 2 * NW) {
                    const int4 e = cv4[kb >> 1];
                    terma(e.x, __int_as_float(e.y));
                    if (kb + 1 < k1) terma(e.z, __int_as_float(e.w));
                }
            } else {
            auto term = [&](int32_t q, float av) -> double {
                double Kv, Jv;
                sums_w(q, Kv, Jv);
                R = __builtin_fma((double)av, Kv, R);
                if (GRAD) Dd = __builtin_fma((double)av, Jv, Dd);
                return Kv;
            };
#pragma unroll
            for (int j = 0; j < FP; ++j) {
                const int32_t kb = 2 * (p0 + NW * j + wv);
                if (kb < k1) {
                    if (kb >= k0) {
                        const double v = term(pr0[j].x, __int_as_float(pr0[j].y));
                        if (SUPP) ks[2 * j] = v;
                    }
                    if (kb + 1 < k1) {
                        const double v = term(pr0[j].z, __int_as_float(pr0[j].w));
                        if (SUPP) ks[2 * j + 1] = v;
                    }
                }
            }
            for (int32_t kb = 2 * (p0 + NW * FP + wv); kb < k1; kb += 2 * NW) {
                const int4 e = cv4[kb >> 1];
                term(e.x, __int_as_float(e.y));
                if (kb + 1 < k1) term(e.z, __int_as_float(e.w));
            }
            }
        if (NW > 1) {
            // the other waves' partial sums to the first, added in wave order
            if (wv > 0) {
                Rs[(wv - 1) * 64 + lane] = R;
                Ds[(wv - 1) * 64 + lane] = Dd;
            }
            __syncthreads();
            if (wv == 0) {
#pragma unroll
                for (int v = 0; v < NW - 1; ++v) {
                    R += Rs[v * 64 + lane];
                    Dd += Ds[v * 64 + lane];
                }
            }
        }
        double t3;
        int m3;
        ld_tm(base + 192, t3, m3);
        // e^{-beta u_i} (anchored records) as the reciprocal of e^{beta u_i}
        // (1 <= e^{beta u_i} <= e^600): a division instead of a second
        // exponential on the first wave, whose share of the batch is the longer
        double ei = 1.0;
        if (anch && valid && wv == 0) ei = recip(eti);
        if (!RM && valid && wv == WE) {
            // compensator terms of the event's node (eq. 2) and their
            // beta-derivative part (eq. 10)
            const double x = bet * (T - ti);
            const double ex = exp_f64(-x);
            // 1 - e^{-x}: by subtraction when every event of the batch has
            // x >= 0.5 (then 1 - e^{-x} >= 0.39 and the subtraction loses
            // nothing), else by expm1 (a wave-uniform choice)
            if (__ballot(x < 0.5) == 0)
                em1 = 1.0 - ex;
            else
                em1 = -expm1(-x);
            const double cs_m = (double)__int_as_float(ni.w);
            comp += cs_m * em1;
            if (GRAD) Esum += cs_m * (T - ti) * ex;
        }
        if (RM && valid && wv == 0) {
            if (anch) {
                R *= ei;
                Dd *= ei;
            }
            rk[i - c0] = R;
            if (GRAD) dk[i - c0] = Dd;
        } else if (valid && wv == 0) {
            if (anch) {
                R *= ei;
                Dd *= ei;
            }
            lam = __builtin_fma(bet, R, (double)__int_as_float(ni.z));
        if (INTENS) lambda_out[i] = (float)lam;
            logsum += log(lam);
            if (GRAD) {
                w = recip(lam);
                gb += w * (R - bet * Dd);
            }
            if (SUPP) {
                // beta w_i K_q(t_i) for each nonzero (m_i, q); the sums past
                // the loaded pairs are formed again
                const double bw = bet * w * ei;
                double* gs = gsup + (int64_t)(s & cmask) * M * M;
#pragma unroll
                for (int j = 0; j < 2 * FP; ++j) {
                    const int32_t k = 2 * p0 + j;
                    if (k >= k0 && k < k1) unsafeAtomicAdd(&gs[k], bw * ks[j]);
                }
                for (int32_t k = 2 * (p0 + FP); k < k1; ++k) {
                    double v, unused;
                    if (anch)
                        sums_a(csr_cv[k].x, v, unused);
                    else
                        sums_w(csr_cv[k].x, v, unused);
                    unsafeAtomicAdd(&gs[k], bw * v);
                }
            }
        }
        if (!RM && GRAD && valid && wv == 0) wchunk[i - c0] = (float)w;
        // the records take the batch's events (wave WC, beside the
        // first wave's work above: nothing there reads the records), then the
        // batch's masks are cleared
        if (anch) {
            // anchored records: the batch's events of a node add their terms,
            // in index order, through one leader lane per node
            if (valid && wv == WC) {
                uint64_t grp = rmask[mi];
                if (__builtin_ctzll(grp) == lane) {
                    const double2 kj = rKJ[mi];
                    double s0 = kj.x, s1 = kj.y;
                    while (grp) {
                        const int j = __builtin_ctzll(grp);
                        grp &= grp - 1;
                        s0 += eb[j];
                        if (GRAD) s1 = __builtin_fma(tb[j] - tref, eb[j], s1);
                    }
                    rKJ[mi] = make_double2(s0, s1);
                }
            }
        } else if (valid && wv == WC) {
            // lazy record update, one leader lane per node, events in index order
            uint64_t grp = rmask[mi];
            if (__builtin_ctzll(grp) == lane) {
                double tq = rtau[mi];
                const double2 kj = rKJ[mi];
                double kq = kj.x, jq = kj.y;
                while (grp) {
                    const int j = __builtin_ctzll(grp);
                    grp &= grp - 1;
                    const double d = tb[j] - tq;
                    const double e = exp_f64(-bet * d);
                    jq = e * __builtin_fma(d, kq, jq);
                    kq = __builtin_fma(e, kq, 1.0);
                    tq = tb[j];
                }
                rtau[mi] = tq;
                rKJ[mi] = make_double2(kq, jq);
            }
        }
        if (wv == WC) {
            lds_wait();   // every lane's read of its mask before the clear
            if (valid) rmask[mi] = 0ull;
        }
        __syncthreads();
        t0 = t1;
        m0 = m1;
        t1 = t2;
        m1 = m2;
        t2 = t3;
        m2 = m3;
        n0 = n1;
        n1 = n2;
#pragma unroll
        for (int j = 0; j < FP; ++j) pr0[j] = pr1[j];
    }
    if (X.bcnt) {
        __syncthreads();
        for (int32_t k = threadIdx.x; k < X.nbo; k += 64 * NW) X.bcnt[(int64_t)k * gridDim.x + s] = lcnt[k];
    }
    // deterministic wave reductions of the float64 partials: the log-sum and
    // dL/dbeta part in the first wave, the compensator sums in wave WE
    if (RM || (wv != 0 && wv != WE)) return;
    for (int off = 32; off > 0; off >>= 1) {
        logsum += __shfl_down(logsum, off, 64);
        comp += __shfl_down(comp, off, 64);
        Esum += __shfl_down(Esum, off, 64);
        gb += __shfl_down(gb, off, 64);
    }
    // the segment slot's sums over the chunks so far (slot s of every chunk,
    // in chunk order; one reduction over the slots ends the call)
    if (lane == 0) {
        double* o = seg_part + (int64_t)s * 4;
        if (wv == 0) {
            o[0] += logsum;
            o[3] += gb;
        }
        if (wv == WE) {
            o[1] += comp;
            o[2] += Esum;
        }
    }
}

// acc[k] += sum over segments of seg_part[s][k] (width values per segment);
// per value a fixed-order tree (deterministic), four values per pass
__global__ __launch_bounds__(256) void large_chunk_acc(int32_t nseg, int32_t width,
                                                       const double* __restrict__ seg_part,
                                                       double* __restrict__ acc) {
    __shared__ double sh[4][256];
    const int tid = threadIdx.x;
    for (int k0 = 0; k0 < width; k0 += 4) {
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (int32_t s = tid; s < nseg; s += 256)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k0 + j < width) v[j] += seg_part[(int64_t)s * width + k0 + j];
#pragma unroll
        for (int j = 0; j < 4; ++j) sh[j][tid] = v[j];
        __syncthreads();
        for (int st = 128; st > 0; st >>= 1) {
            if (tid < st)
#pragma unroll
                for (int j = 0; j < 4; ++j) sh[j][tid] += sh[j][tid + st];
            __syncthreads();
        }
        if (tid < 4 && k0 + tid < width) acc[k0 + tid] += sh[tid][0];
        __syncthreads();
    }
}

// Several decay kernels (Background, eq. 1 with K > 1): the per-kernel
// forward passes left R_k(i) = alpha^k_{m_i,:} . K^k(t_i) and D_k(i) =
// alpha^k_{m_i,:} . J^k(t_i) for each event of the chunk; here
//   lambda_i = mu_{m_i} + sum_k beta_k R_k(i),   w_i = 1 / lambda_i,
// and the segment's float64 partials: log-sum, compensator
// sum_k colsum_k[m_i] (1 - e^{-beta_k (T - t_i)}), and per kernel E_k (its
// beta-derivative) and sum_i w_i (R_k(i) - beta_k D_k(i)) (eq. 10 per kernel).
// One workgroup of 256 per segment, fixed-order block sums, added to the
// segment slot's sums over the chunks so far (as in large_forward).
template <bool GRAD, bool INTENS>
__global__ __launch_bounds__(256) void large_combine(int64_t c0, int64_t c1, int32_t M, int32_t K, double T,
                                                     const double* __restrict__ t,
                                                     const int32_t* __restrict__ marks,
                                                     const float* __restrict__ mu, const float* __restrict__ beta,
                                                     const float* __restrict__ colsum,
                                                     const double* __restrict__ rk, const double* __restrict__ dk,
                                                     int64_t CH, double* __restrict__ seg_part,
                                                     float* __restrict__ wchunk, float* __restrict__ lambda_out) {
    __shared__ double sh[256];
    const int32_t s = blockIdx.x;
    const int64_t a = c0 + (int64_t)s * HK_SEG;
    const int64_t b = a + HK_SEG < c1 ? a + HK_SEG : c1;
    double logsum = 0.0, comp = 0.0, E[HK_KMAX], gb[HK_KMAX];
#pragma unroll
    for (int k = 0; k < HK_KMAX; ++k) E[k] = gb[k] = 0.0;
    for (int64_t i = a + threadIdx.x; i < b; i += 256) {
        const int mi = clamp_mark(marks[i], M);
        const double ti = t[i];
        const int64_t r = i - c0;
        double lam = (double)mu[mi];
        for (int k = 0; k < K; ++k) lam = __builtin_fma((double)beta[k], rk[k * CH + r], lam);
        if (INTENS) lambda_out[i] = (float)lam;
        logsum += log(lam);
        const double w = 1.0 / lam;
        if (GRAD) wchunk[r] = (float)w;
#pragma unroll
        for (int k = 0; k < HK_KMAX; ++k) {
            if (k < K) {
                const double bk = (double)beta[k];
                const double x = bk * (T - ti);
                const double cs = (double)colsum[(int64_t)k * M + mi];
                comp += cs * -expm1(-x);
                if (GRAD) {
                    E[k] += cs * (T - ti) * exp_f64(-x);
                    gb[k] += w * (rk[k * CH + r] - bk * dk[k * CH + r]);
                }
            }
        }
    }
    const int W = 2 + 2 * K;
    double* o = seg_part + (int64_t)s * W;
    double v = block_sum_d<256>(logsum, sh);
    if (threadIdx.x == 0) o[0] += v;
    v = block_sum_d<256>(comp, sh);
    if (threadIdx.x == 0) o[1] += v;
#pragma unroll
    for (int k = 0; k < HK_KMAX; ++k) {
        if (k < K) {
            v = block_sum_d<256>(E[k], sh);
            if (threadIdx.x == 0) o[2 + k] += v;
            v = block_sum_d<256>(gb[k], sh);
            if (threadIdx.x == 0) o[2 + K + k] += v;
        }
    }
}

// ------------------------------------------------------------------ finalize
// Final sums, blockIdx.z = kernel k of K (decay kernels): the log-likelihood and
// dL/dmu with k = 0, dL/dbeta, dL/dalpha from the partials.  The call-level
// sums (logsum, comp, E[K], gbeta[K]) are those of the nslot segment slots
// seg_part[nslot][2 + 2K], summed here by a fixed tree, or (seg_part null) acc;
// ebacc: per-target decays, dL/dbeta = -ebacc, else null.
// Every entry is summed over ER partials of dL/dalpha, and its column over NSC
// partials of the weights and compensator terms, each in a fixed order: a
// workgroup takes CB columns and FR rows, its SR = 256 / CB thread rows are ES
// slices of the partials times SR / ES matrix rows, slice sums are added by a
// tree.  Bound by the read of the partials; with one thread per entry the 512
// partials of a 16-node model were a chain of dependent loads (n = 1e6:
// 123 us, and 35 us more for the column sums, against 10 us now).
// CB = 16; 64 for many nodes with few partials (ES = 1): rows of alpha then start
// anywhere in a cache line, and strips of 16 columns write two halves of lines
// each (M = 6700, one range: 180 us with 64 columns, 228 with 16; M = 6000: 113,
// in tiles of 16 x 16 entries 216).
template <int SR, int CB>
__device__ __forceinline__ double fin_tree(double v, double (*sh)[CB + 1], int c, int s, int w) {
    // sum of v over the w slices of this thread's group (w a power of two,
    // groups of w consecutive s), returned to the group's first slice
    sh[s][c] = v;
    __syncthreads();
    for (int h = w >> 1; h > 0; h >>= 1) {
        if ((s & (w - 1)) < h) sh[s][c] += sh[s + h][c];
        __syncthreads();
    }
    const double r = sh[s][c];
    __syncthreads();
    return r;
}

template <int CB>
__global__ __launch_bounds__(256) void large_final(int32_t M, int32_t ER, int32_t NSC, int32_t ES, double T,
                                                   const float* __restrict__ mu, const double* __restrict__ seg_part,
                                                   int32_t nslot, const double* __restrict__ acc,
                                                   const double* __restrict__ ebacc, const double* __restrict__ gpart,
                                                   const double* __restrict__ spart,
                                                   const double* __restrict__ cpart, double* __restrict__ loglik,
                                                   double* __restrict__ g_mu, double* __restrict__ g_alpha,
                                                   double* __restrict__ g_beta, double* __restrict__ csum, int grad,
                                                   int32_t K, int32_t NSP, int32_t FR) {
    constexpr int SR = 256 / CB;
    __shared__ double sh[SR][CB + 1];
    __shared__ double ps[256];
    const int64_t MM = (int64_t)M * M;
    const int c = threadIdx.x & (CB - 1), s = threadIdx.x / CB;
    const int32_t k = blockIdx.z;
    if (gpart) gpart += (int64_t)k * ER * MM;
    if (grad) {
        spart += (int64_t)k * NSP * M;
        cpart += (int64_t)k * NSP * M;
        if (g_alpha) g_alpha += (int64_t)k * MM;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        // sums in a fixed order: strided partial sums, then a tree
        auto total = [&](double v) {
            ps[threadIdx.x] = v;
            __syncthreads();
            for (int h = 128; h > 0; h >>= 1) {
                if ((int)threadIdx.x < h) ps[threadIdx.x] += ps[threadIdx.x + h];
                __syncthreads();
            }
            const double r = ps[0];
            __syncthreads();
            return r;
        };
        double v = 0.0;
        for (int32_t p = threadIdx.x; p < M; p += 256) v += (double)mu[p];
        const double musum = total(v);
        const int32_t W = 2 + 2 * K;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        if (seg_part) {
#pragma unroll 4
            for (int32_t i = threadIdx.x; i < nslot; i += 256) {
                const double* o = seg_part + (int64_t)i * W;
                a0 += o[0];
                a1 += o[1];
                a2 += o[2 + k];
                a3 += o[2 + K + k];
            }
            a0 = total(a0);
            a1 = total(a1);
            a2 = total(a2);
            a3 = total(a3);
        } else {
            a0 = acc[0];
            a1 = acc[1];
            a2 = acc[2 + k];
            a3 = acc[2 + K + k];
        }
        if (threadIdx.x == 0) {
            if (k == 0) loglik[0] = a0 - T * musum - a1;
            if (grad && g_beta && !ebacc) g_beta[k] = a3 - a2;
        }
    }
    if (!grad) return;
    const int32_t q = blockIdx.x * CB + c;
    const int32_t qc = q < M ? q : M - 1;
    // the columns' compensator sums (every workgroup of the columns), dL/dmu
    // and the per-target dL/dbeta (the first)
    double cs = 0.0;
#pragma unroll 8
    for (int32_t e = s; e < NSC; e += SR) cs += cpart[(int64_t)e * M + qc];
    cs = fin_tree<SR, CB>(cs, sh, c, s, SR);
    if (s == 0) ps[c] = cs;
    __syncthreads();
    cs = ps[c];
    if (blockIdx.y == 0) {
        if (k == 0) {
            double v = 0.0;
#pragma unroll 8
            for (int32_t e = s; e < NSC; e += SR) v += spart[(int64_t)e * M + qc];
            v = fin_tree<SR, CB>(v, sh, c, s, SR);
            if (s == 0 && q < M && g_mu) g_mu[q] = v - T;
        }
        if (s == 0 && q < M) {
            if (ebacc && g_beta) g_beta[q] = -ebacc[q];
            if (csum) csum[q] = cs;
        }
    }
    if (!g_alpha) return;
    const int rw = SR / ES, es = s & (ES - 1);
    if (ES == 1) {
        // a thread an entry of each row: the rows' loads side by side
#pragma unroll 4
        for (int32_t r0 = 0; r0 < FR; r0 += SR) {
            const int32_t row = blockIdx.y * FR + r0 + s;
            if (row < M && q < M) {
                const int64_t x = (int64_t)row * M + q;
                double g = 0.0;
                if (gpart)
                    for (int32_t e = 0; e < ER; ++e) g += gpart[(int64_t)e * MM + x];
                // gpart null: zero (large_sup_scatter then writes the support)
                g_alpha[x] = gpart ? g - cs : 0.0;
            }
        }
        return;
    }
    for (int32_t r0 = 0; r0 < FR; r0 += rw) {
        const int32_t row = blockIdx.y * FR + r0 + s / ES;
        const int32_t rc = row < M ? row : M - 1;
        const int64_t x = (int64_t)rc * M + qc;
        double g = 0.0;
        if (gpart) {
#pragma unroll 8
            for (int32_t e = es; e < ER; e += ES) g += gpart[(int64_t)e * MM + x];
        }
        g = fin_tree<SR, CB>(g, sh, c, s, ES);
        if (es == 0 && row < M && q < M) g_alpha[x] = gpart ? g - cs : 0.0;
    }
}

void large_final_launch(const LargeArgs& A, bool slots, const double* ebacc, const double* gpart, double* csum,
                        hipStream_t st) {
    // slices of the partials: enough that a slice sums at most about 8, as
    // long as that leaves a slice several
    int32_t ES = 1;
    while (ES < 16 && A.ER > 8 * ES) ES <<= 1;
    // rows per workgroup: 16, or one pass of its thread rows where that leaves
    // the chip idle (few nodes); more with many nodes, so that a workgroup's
    // column sums are made for more than a tile
    const int32_t M = A.M;
    const bool wide = ES == 1 && M >= 1024;
    const unsigned gx = (unsigned)(wide ? (M + 63) / 64 : (M + 15) / 16);
    int32_t FR = (int64_t)gx * gx < 256 && !wide ? 16 / ES : 16;
    while ((int64_t)gx * (M / FR) > 8192) FR <<= 1;
    const unsigned gy = (unsigned)((M + FR - 1) / FR);
    const unsigned gz = (unsigned)A.K;
    auto go = [&](auto* kern) {
        hipLaunchKernelGGL(kern, A.grad ? dim3(gx, A.g_alpha ? gy : 1, gz) : dim3(1), dim3(256), 0, st, M, A.ER,
                           A.ER, ES, A.T, A.mu, slots ? A.seg_part : (const double*)nullptr, A.nseg, A.acc, ebacc,
                           gpart, A.spart, A.cpart_, A.loglik, A.g_mu, A.g_alpha, A.g_beta, csum, A.grad ? 1 : 0,
                           A.K, A.NSP, FR);
    };
    if (wide)
        go(large_final<64>);
    else
        go(large_final<16>);
}

// support-restricted dL/dalpha: one wave per row p writes, for each nonzero
// (p, q) of alpha, the first term summed over the ncopy copies (in order)
// minus the column's compensator sum (csum, from large_final); runs after
// large_final zeroed g_alpha
__global__ __launch_bounds__(64) void large_sup_scatter(int32_t M, int32_t ncopy,
                                                        const int32_t* __restrict__ csr_ptr,
                                                        const int2* __restrict__ csr_cv,
                                                        const double* __restrict__ gsup,
                                                        const double* __restrict__ csum,
                                                        double* __restrict__ g_alpha) {
    const int32_t p = blockIdx.x;
    const int64_t MM = (int64_t)M * M;
    const int32_t k1 = csr_ptr[p + 1];
    for (int32_t k = csr_ptr[p] + (int32_t)threadIdx.x; k < k1; k += 64) {
        const int32_t q = csr_cv[k].x;
        double g = 0.0;
        for (int32_t c = 0; c < ncopy; ++c) g += gsup[c * MM + k];
        g_alpha[(int64_t)p * M + q] = g - csum[q];
    }
}

// ------------------------------------------------------------------ host
static void large_rules(LargeArgs& A, const hawkes_problem* p, const hawkes_tuning& tu) {
    A.n = p->n;
    A.M = p->m;
    A.K = p->k;
    A.per_target = p->beta_mode == HAWKES_BETA_PER_TARGET;
    A.T = p->T;
    // chunks no longer than the sequence needs (at least 2^12 events): the
    // per-chunk buffers then scale with n for short sequences
    int lg = p->chunk_log2 ? p->chunk_log2 : 20;
    while (lg > 12 && ((int64_t)1 << (lg - 1)) >= p->n) --lg;
    // a record of the per-target dense kernel: the event's index in the chunk
    // beside the 7 bits of its node in the block
    if (A.per_target && lg > 25) lg = 25;
    A.CH = (int64_t)1 << lg;
    A.nchunks = (A.n + A.CH - 1) / A.CH;
    // per-target decays, few events: shorter segments, about 1024 of them (one
    // wave each in the aggregation and the forward pass; n = 2e5, M = 100:
    // 54 + 31 us with 256 events, 173 + 96 with 1024)
    A.seg = HK_SEG;
    if (A.per_target && A.M <= 1024)
        while (A.seg > HK_PT_SEG_MIN && (A.n < A.CH ? A.n : A.CH) < (int64_t)1024 * A.seg &&
               (A.CH / A.seg) * 2 * A.M <= HK_PT_SEG_ROWS)
            A.seg >>= 1;
    A.nseg = (int32_t)((A.CH + A.seg - 1) / A.seg);
    A.NB = (A.M + HK_PT_NB - 1) / HK_PT_NB;
    // few nodes, one kernel: hk_narrow.hip, up to the 64 lanes of a wave.  The
    // forward pass, partition and dense kernels against it, n = 1e6: M = 16:
    // 87 + 14 + 86 us against 44; M = 50, dense rows: 119 + 13 + 119 against 95
    A.narrow = !A.per_target && A.K == 1 && A.M <= HK_NARROW_MAX_M;
    if (A.narrow) {
        // workgroups (each with its partial sums), two segments a round: two
        // a CU where the sequence has that many.  dense_ranges does not apply: it
        // would bound the workgroups of the whole pass, log-likelihood and
        // intensities included
        const int64_t segs = A.n < A.CH ? (A.n + HK_SEG - 1) / HK_SEG : A.nseg;
        const int64_t er = (segs + 1) / 2 < 512 ? (segs + 1) / 2 : 512;
        A.ER = er < 1 ? 1 : (int32_t)er;
    } else if (A.per_target) {
        // Event ranges of the per-target dense kernel, one workgroup a CU at a
        // time: the number whose rounds of 256 workgroups take least, a
        // workgroup 18 ns for each of its source block's events (measured at
        // M = 4096) and 22 us beside them, a range the traffic of its partials
        // (both set by calls of 1 to 4 ranges, us: M = 2100, 2e5 events 915 /
        // 840 / 828 / 869, 6e4 events 598 / 608 / 625 / 646; M = 1450, 2e5
        // 741 / 760 / 678 / 711; M = 3000, 3e5 1507 / 1479 / 1485 / 1565, all
        // with the first chunk's partials cleared and read, 10 to 50 us more);
        // with some events for every wave and about 256 MiB of partials at most.
        const int64_t ev = A.n < A.CH ? A.n : A.CH, nbb = (int64_t)A.NB * A.NB;
        int64_t most = ev / (HK_PT_WAVE_EV * 16);
        const int64_t fit = ((int64_t)256 << 20) / ((int64_t)A.M * A.M * 8);
        if (most > fit && fit >= 256 / nbb) most = fit;   // (one round's ranges always)
        const int64_t few = 768 / nbb > 8 ? 768 / nbb : 8;   // up to three rounds, or eight ranges
        if (most > few) most = few;
        double best = 0.0;
        A.ER = 1;
        for (int64_t er = 1; er <= most; ++er) {
            const double cost = (double)((nbb * er + 255) / 256) *
                                    (0.018 * (double)ev / (double)(A.NB * er) + 22.0) +
                                (double)er * 12.0 * (double)A.M * (double)A.M / 4.5e6;
            if (er == 1 || cost < best) {
                best = cost;
                A.ER = (int32_t)er;
            }
        }
        A.BL = 6;
    } else {
        // dense dL/dalpha (hk_dense.hip)
        // rows of U and K, and their product, in float32 from HK_F32_MIN_M nodes
        // on; in float64 on chunks above 2^24 events and where a caller sets
        // dense_cols to 64 or 128 or dense_rows to 16
        A.row64 = A.M < HK_F32_MIN_M || lg > 24 || tu.dense_cols == 64 || tu.dense_cols == 128 || tu.dense_rows == 16;
        // tiles of 16 rows x up to 1024 columns (128 KiB of LDS; 384 with
        // float64 rows, whose product holds twice the registers a column): one
        // column block, or several of a multiple of 64 columns
        const int32_t widest = A.row64 ? HK_CW64 : 1024;
        A.NCB = (A.M + widest - 1) / widest;
        if (A.NCB == 1) {
            // events per block: the pair terms cost half a block of records per
            // event, the product M^2 multiply-adds per block.  dense_prep +
            // dense_tiles, us a launch with 64 / 128 / 256 events: M = 50, n =
            // 1e6: 119 / 142 / 208; M = 251, n = 3e5: 54 / 49 / 58; M = 700, 2^20:
            // - / 223 / 203; M = 1000, 2^20: - / 335 / 215 (an earlier form)
            A.BL = A.M > 512 ? 8 : A.M > 128 ? 7 : 6;
            if (tu.dense_cols > 0) A.BL = tu.dense_cols == 256 ? 8 : tu.dense_cols == 128 ? 7 : 6;
            // few nodes: each has several columns of the tile, which its records
            // take in turn (64 records on one address are added one by one: K =
            // 2, M = 1, 3e6 events 3892 us a call with one column, 2486 now)
            A.rep = 1;
            while (2 * A.rep * A.M <= 64) A.rep <<= 1;
            A.CW = (A.M * A.rep + 15) & ~15;
        } else {
            // several column blocks: an event meets half a block's records of
            // each of them, so longer blocks (us a call with 256 / 512 / 1024
            // events, n = 1e6: M = 1025: 625 / 541 / 743; 2048: 713 / 529 / 555;
            // 2200: 1092 / 744 / 656; 4096: 2496 / 1487 / 1048; float64 rows, M =
            // 512: 284 / 283 / 410; 1000: 636 / 499 / 627; 1500: 1023 / 724 / 643;
            // 4096: 5094 / 2846 / 1895).  Tuned: for dense_cols = 64 and 128 half
            // the rule's, for 256 at least 512.
            A.BL = A.M > (A.row64 ? 1152 : 2048) ? 10 : A.M > 512 ? 9 : 8;
            if (tu.dense_cols == 256 && A.BL < 9) A.BL = 9;
            if ((tu.dense_cols == 64 || tu.dense_cols == 128) && A.BL > 8) --A.BL;
            A.rep = 1;
            A.CW = (((A.M + A.NCB - 1) / A.NCB) + 63) & ~63;
        }
        A.DRB = 4;
        A.NBO = (A.M + 15) >> 4;
        // event ranges: one round of workgroups (one a CU), and at least two
        // blocks for every wave
        const int64_t blks = ((A.n < A.CH ? A.n : A.CH) >> A.BL) + 1;
        int64_t er = 256 / ((int64_t)A.NBO * A.NCB);
        if (er > blks / 24) er = blks / 24;
        // and about 32 MiB of partials
        const int64_t most = ((int64_t)32 << 20) / ((int64_t)A.K * A.M * A.M * 8);
        if (er > 4 && er > most) er = most > 4 ? most : 4;
        if (tu.dense_ranges > 0) {
            er = tu.dense_ranges;
            while (er > A.nseg) er >>= 1;
        }
        A.ER = er < 1 ? 1 : (int32_t)er;
    }
    // rows of the sums per node: one a range; room for 16 where they are small
    // beside the dL/dalpha partials (one kernel, one column block or float64
    // rows), so that there the workspace of up to 16 ranges differs by the
    // dL/dalpha partials alone
    A.NSP = A.ER < 16 && !A.per_target && !A.narrow && A.K == 1 && (A.NCB == 1 || A.row64) ? 16 : A.ER;
    A.Mp = (A.M + 63) & ~63;
}

// carves the workspace of A's choices; its size (pointers with ws not null)
static size_t large_carve(LargeArgs& A, bool grad, void* ws, size_t ws_bytes) {
    A.grad = grad;
    const int64_t M = A.M, MM = M * M, K = A.K;
    Carve c(ws, ws_bytes);
    A.csr_ptr = c.take<int32_t>(K * (M + 1));
    A.csr_cv = c.take<int2>(K * cv_stride(MM));
    A.colsum = c.take<float>(K * M);
    A.rcnt = c.take<int32_t>(K * M);
    if (K > 1) {
        A.rk = c.take<double>((size_t)K * A.CH);
        if (grad) A.dk = c.take<double>((size_t)K * A.CH);
    }
    A.agg = c.take<double>((size_t)A.nseg * 2 * M);
    A.seg_span = c.take<double>(A.nseg);
    A.seg_dec = c.take<double>(A.nseg);
    A.seg_off = c.take<double>(A.nseg);
    A.seg_offdec = c.take<double>(A.nseg);
    A.ngr = (A.nseg + HK_SG - 1) / HK_SG;
    A.gagg = c.take<double>((size_t)A.ngr * 2 * M);
    A.gcarry = c.take<double>((size_t)A.ngr * 2 * M);
    A.gspan = c.take<double>(A.ngr);
    A.gdec = c.take<double>(A.ngr);
    A.node_info = c.take<int4>(K * M);
    A.carry_seg = c.take<double>((size_t)K * A.nseg * 2 * M);
    A.carry = c.take<double>(K * 2 * M);
    A.pt_flags = c.take<float>(2);
    A.seg_part = c.take<double>((size_t)A.nseg * (2 + 2 * K));
    A.acc = c.take<double>(2 + 2 * K);
    A.ll_scratch = c.take<double>(1);
    if (grad && !A.per_target) A.csum = c.take<double>(M);
    if (A.per_target) {
        A.csc_ptr = c.take<int32_t>(M + 1);
        A.csc_cv = c.take<int2>(MM);
        A.ebseg = c.take<double>((size_t)A.nseg * M);
        A.ebacc = c.take<double>(M);
        if (grad) {
            // constant memory: w of one chunk, and two levels of chunk-start
            // states (the chunks of each level-1 slot are chained again into
            // the level-2 slots during the reverse sweep)
            A.wv = c.take<float>((size_t)A.CH);
            A.pt_ckr = (A.nchunks + HK_PTCK - 1) / HK_PTCK;
            if (A.pt_ckr < 1) A.pt_ckr = 1;
            A.pt_ck = c.take<double>((size_t)2 * HK_PTCK * 2 * M);
            A.aggA = c.take<double>((size_t)A.nseg * M);
            A.rcarry_seg = c.take<double>((size_t)A.nseg * M);
            A.rgagg = c.take<double>((size_t)A.ngr * M);
            A.rgcarry = c.take<double>((size_t)A.ngr * M);
            A.achunk = c.take<double>(M);
        }
    }
    if (grad) {
        if (!A.per_target && !A.narrow) A.wchunk = c.take<float>(A.CH);
        if (A.per_target) {
            A.bk_cnt = c.take<int32_t>((size_t)A.NB * A.nseg);
            A.bk_off = c.take<int32_t>((size_t)A.NB * (A.nseg + 1));
            A.bk_base = c.take<int32_t>(A.NB);
            A.bk_key = c.take<uint32_t>(A.CH);
            A.bk_t = c.take<double>(A.CH);
            A.bk_w = c.take<float>(A.CH);
        }
        A.gpart = c.take<double>((size_t)K * A.ER * MM);
        A.spart = c.take<double>((size_t)K * A.NSP * M);
        A.cpart_ = c.take<double>((size_t)K * A.NSP * M);
        if (!A.per_target && !A.narrow) {
            const size_t rows = (size_t)(A.CH >> A.BL) * A.Mp + 1024;
            A.urow = c.take<double>(A.row64 ? rows : rows / 2);
            A.krow = c.take<double>(A.row64 ? rows : rows / 2);
            A.prec = c.take<uint2>(A.NCB > 1 ? (size_t)(A.CH >> A.BL) * HK_LSLOTS(A.BL, A.NCB) : (size_t)A.CH);
            if (A.NCB > 1) A.plist = c.take<int32_t>((size_t)(A.CH >> A.BL) * (A.NCB + 1));
            A.wide = c.take<int32_t>(A.CH >> A.BL);
            A.bo_cnt = c.take<int32_t>((size_t)A.NBO * A.nseg);
            A.bo_off = c.take<int32_t>((size_t)A.NBO * (A.nseg + 1));
            A.bo_base = c.take<int32_t>(A.NBO);
            A.bo_key = c.take<uint32_t>(A.CH);
            A.bo_cw = c.take<float2>(A.CH);
            A.bo_e = c.take<double>(A.CH);
        }
    }
    return c.off + 256;
}

size_t large_layout(LargeArgs& A, const hawkes_problem* p, bool grad, void* ws, size_t ws_bytes, size_t fit) {
    const hawkes_tuning tu = tuning_snapshot();
    large_rules(A, p, tu);
    const bool tuned = tu.dense_ranges > 0 || tu.dense_cols > 0 || tu.dense_rows > 0;
    if (fit > 0 && grad && !A.narrow && !A.per_target &&
        large_carve(A, true, nullptr, 0) > fit) {
        // no spare rows of the sums per node; with the dense kernels tuned longer
        // blocks, then fewer ranges, then (not far above) the same with chunks
        // half as long
        hawkes_problem h = *p;
        LargeArgs B = A;
        for (int pass = 0; pass < 2; ++pass) {
            for (;;) {
                B.NSP = B.ER;
                if (large_carve(B, true, nullptr, 0) <= fit) {
                    A = B;
                    return large_carve(A, true, ws, ws_bytes);
                }
                if (!tuned)
                    break;
                else if (B.BL < (B.NCB > 1 ? 10 : 8))
                    ++B.BL;
                else if (B.ER > 1)
                    B.ER >>= 1;
                else
                    break;
            }
            h.chunk_log2 = 0;
            while (((int64_t)2 << h.chunk_log2) < A.CH) ++h.chunk_log2;
            if (!tuned || h.chunk_log2 < 12 || large_carve(B, true, nullptr, 0) > fit + fit / 2) break;
            B = A;
            large_rules(B, &h, tu);
        }
    }
    return large_carve(A, grad, ws, ws_bytes);
}

void large_chunk_acc_launch(int32_t nseg, int32_t width, const double* seg_part, double* acc, hipStream_t st) {
    hipLaunchKernelGGL(large_chunk_acc, dim3(1), dim3(256), 0, st, nseg, width, seg_part, acc);
}

size_t lds_limit() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 64 * 1024;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
        return 64 * 1024;
    return (size_t)v;
}

// Kernels whose dynamic LDS exceeds 64 KiB are allowed, once per (kernel,
// device), as much as the device's per-workgroup LDS leaves beside the
// kernel's own static LDS (asking for more than that is refused); later calls
// (including ones under stream capture) only look the pair up.  A refusal
// clears the runtime's last-error state, so that it does not surface at an
// unrelated later call.
hawkes_status allow_lds(const void* kernel, size_t bytes, bool with_static) {
    const size_t lim = lds_limit();
    if (bytes > lim) return HAWKES_EUNSUPPORTED;
    // with_static: the kernel's static LDS comes on top of `bytes`, so the
    // grant is needed even at 64 KiB of dynamic LDS
    if (!with_static && bytes <= 64 * 1024) return HAWKES_OK;
    static std::mutex mu;
    static const void* done_k[128];
    static int done_d[128];
    static size_t done_cap[128];
    static int n_done = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return HAWKES_EDEVICE;
    std::lock_guard<std::mutex> g(mu);
    for (int i = 0; i < n_done; ++i)
        if (done_k[i] == kernel && done_d[i] == dev) return bytes <= done_cap[i] ? HAWKES_OK : HAWKES_EUNSUPPORTED;
    hipFuncAttributes fa;
    if (hipFuncGetAttributes(&fa, kernel) != hipSuccess) {
        (void)hipGetLastError();
        return HAWKES_EDEVICE;
    }
    if (fa.sharedSizeBytes >= lim) return HAWKES_EUNSUPPORTED;
    const size_t cap = lim - fa.sharedSizeBytes;
    if (bytes > cap) return HAWKES_EUNSUPPORTED;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)cap) != hipSuccess) {
        (void)hipGetLastError();
        return HAWKES_EUNSUPPORTED;
    }
    if (n_done < 128) {
        done_k[n_done] = kernel;
        done_d[n_done] = dev;
        done_cap[n_done] = cap;
        ++n_done;
    }
    return HAWKES_OK;
}

void large_scan(LargeArgs& A, int32_t nseg, const float* beta_pt, hipStream_t st, bool apply) {
    const int32_t M = A.M;
    // the first two passes are serial chains per thread, ngr * M and M
    // threads in all: workgroups of one wave spread them over every CU
    const unsigned gM = (unsigned)((M + 63) / 64);
    const int32_t ngr = (nseg + HK_SG - 1) / HK_SG;
    const int64_t nloc = (int64_t)ngr * M, napp = (int64_t)nseg * M;
    hipLaunchKernelGGL(large_scan_local, dim3((unsigned)((nloc + 63) / 64)), dim3(64), 0, st, nseg, M, A.agg,
                       A.seg_dec, A.seg_span, A.carry_seg, A.gagg, beta_pt, A.beta, A.gspan, A.gdec, A.seg_off,
                       A.seg_offdec);
    hipLaunchKernelGGL(large_scan_groups, dim3(gM), dim3(64), 0, st, nseg, M, A.gagg, A.gspan, A.gdec, A.gcarry,
                       A.carry, beta_pt);
    if (apply)
        hipLaunchKernelGGL(large_scan_apply, dim3((unsigned)((napp + 255) / 256)), dim3(256), 0, st, nseg, M,
                           A.seg_off, A.seg_offdec, A.gcarry, A.carry_seg, beta_pt);
}

// the dense gradient's partials of a sequence without events (otherwise the
// first chunk stores them)
static void dense_zero(const LargeArgs& A, ZeroList& Z) {
    Z.add(A.gpart, (int64_t)A.K * A.ER * A.M * A.M);
    Z.add(A.spart, (int64_t)A.K * A.NSP * A.M);
    Z.add(A.cpart_, (int64_t)A.K * A.NSP * A.M);
}

// launches the forward pass's form of four waves per segment, or of two
template <bool GRAD, bool INTENS, bool RM>
struct Fwd {
    static const void* kernel(int32_t M) {
        return M <= HK_FW4_MAX_M ? (const void*)large_forward<GRAD, INTENS, false, 4, RM>
                                 : (const void*)large_forward<GRAD, INTENS, false, 2, RM>;
    }
    template <typename... Args>
    static void launch(int32_t M, int32_t nseg, size_t lds, hipStream_t st, Args... args) {
        if (M <= HK_FW4_MAX_M)
            hipLaunchKernelGGL((large_forward<GRAD, INTENS, false, 4, RM>), dim3(nseg), dim3(256), lds, st, args...);
        else
            hipLaunchKernelGGL((large_forward<GRAD, INTENS, false, 2, RM>), dim3(nseg), dim3(128), lds, st, args...);
    }
};

// Several decay kernels (K > 1, shared decay per kernel; Background eq. 1,
// gradients per kernel as in eqs. 8-10).  Per chunk: for each kernel k its
// segment maps, carries and forward pass (R mode), then large_combine forms
// lambda and the shared w_i = 1/lambda_i; with the gradient the chunk's events
// are partitioned once and the dense dL/dalpha kernels run once per kernel
// (decay beta_k, kernel k's state rows and partial sums).
static hawkes_status run_large_multi(LargeArgs& A, hipStream_t st) {
    const int32_t M = A.M, K = A.K;
    const int64_t MM = (int64_t)M * M;
    const size_t lds_agg = (size_t)2 * M * sizeof(double);
    const size_t lds_fwd = (size_t)M * (sizeof(uint64_t) + 2 * sizeof(double));
    if (allow_lds((const void*)large_seg_agg, lds_agg) != HAWKES_OK ||
        allow_lds(Fwd<true, false, true>::kernel(M), lds_fwd) != HAWKES_OK ||
        allow_lds(Fwd<false, false, true>::kernel(M), lds_fwd) != HAWKES_OK)
        return HAWKES_EUNSUPPORTED;
    if (A.grad && dense_allow_lds(A) != HAWKES_OK) return HAWKES_EUNSUPPORTED;
    const int32_t W = 2 + 2 * K;
    // cleared: the carried states and the segment slots' sums over the chunks
    ZeroList Z{};
    Z.add(A.carry, (int64_t)K * 2 * M);
    Z.add(A.seg_part, (int64_t)A.nseg * W);
    if (A.grad && A.nchunks == 0) dense_zero(A, Z);
    // column sums, CSR copies and node records of every alpha^k
    large_setup_launch(A, 0, true, true, Z, st);
    large_index_launch(A, 0, A.csr_ptr, A.csr_cv, A.node_info, nullptr, st);
    // kernel k's view of the per-kernel arrays
    auto view = [&](int32_t k) {
        LargeArgs B = A;
        B.K = 1;
        B.beta = A.beta + k;
        B.carry = A.carry + (int64_t)k * 2 * M;
        B.carry_seg = A.carry_seg + (int64_t)k * A.nseg * 2 * M;
        B.gpart = A.gpart ? A.gpart + (int64_t)k * A.ER * MM : nullptr;
        B.spart = A.spart ? A.spart + (int64_t)k * A.NSP * M : nullptr;
        B.cpart_ = A.cpart_ ? A.cpart_ + (int64_t)k * A.NSP * M : nullptr;
        return B;
    };
    for (int64_t ch = 0; ch < A.nchunks; ++ch) {
        const int64_t c0 = ch * A.CH;
        const int64_t c1 = c0 + A.CH < A.n ? c0 + A.CH : A.n;
        const int32_t nseg = (int32_t)((c1 - c0 + HK_SEG - 1) / HK_SEG);
        for (int32_t k = 0; k < K; ++k) {
            LargeArgs B = view(k);
            // the lazy records' times go to the segment maps' buffer, which
            // the scan has consumed by then
            FwdExtra Xm{};
            Xm.rtau = B.agg;
            {
                TimedScope ts(2, st);
                hipLaunchKernelGGL(large_seg_agg, dim3(nseg), dim3(64), lds_agg, st, c0, c1, M, A.t, A.marks,
                                   B.beta, B.agg, B.seg_span, B.seg_dec);
            }
            {
                TimedScope ts(3, st);
                large_scan(B, nseg, nullptr, st);
            }
            TimedScope ts(1, st);
            if (A.grad)
                Fwd<true, false, true>::launch(M, nseg, lds_fwd, st, c0, c1, M, A.T, A.t, A.marks, A.mu, B.beta,
                                   A.node_info + (int64_t)k * M, A.csr_cv + k * cv_stride(MM), B.carry_seg,
                                   A.seg_part, A.wchunk, (float*)nullptr, (double*)nullptr, 0,
                                   A.rk + (int64_t)k * A.CH, A.dk + (int64_t)k * A.CH, Xm);
            else
                Fwd<false, false, true>::launch(M, nseg, lds_fwd, st, c0, c1, M, A.T, A.t, A.marks, A.mu, B.beta,
                                   A.node_info + (int64_t)k * M, A.csr_cv + k * cv_stride(MM), B.carry_seg,
                                   A.seg_part, A.wchunk, (float*)nullptr, (double*)nullptr, 0,
                                   A.rk + (int64_t)k * A.CH, (double*)nullptr, Xm);
        }
        {
            TimedScope ts(1, st);
            if (A.grad)
                hipLaunchKernelGGL((large_combine<true, false>), dim3(nseg), dim3(256), 0, st, c0, c1, M, K, A.T, A.t,
                                   A.marks, A.mu, A.beta, A.colsum, A.rk, A.dk, A.CH, A.seg_part, A.wchunk,
                                   (float*)nullptr);
            else if (A.lambda_out)
                hipLaunchKernelGGL((large_combine<false, true>), dim3(nseg), dim3(256), 0, st, c0, c1, M, K, A.T, A.t,
                                   A.marks, A.mu, A.beta, A.colsum, A.rk, A.dk, A.CH, A.seg_part, A.wchunk,
                                   A.lambda_out);
            else
                hipLaunchKernelGGL((large_combine<false, false>), dim3(nseg), dim3(256), 0, st, c0, c1, M, K, A.T,
                                   A.t, A.marks, A.mu, A.beta, A.colsum, A.rk, A.dk, A.CH, A.seg_part, A.wchunk,
                                   (float*)nullptr);
        }
        if (A.grad) {
            {
                TimedScope tb(6, st);
                bucket_starts(A, c0, c1, nseg, A.DRB, A.bo_cnt, A.bo_off, st, false);
            }
            for (int32_t k = 0; k < K; ++k) {
                LargeArgs B = view(k);
                large_dense_launch(B, c0, c1, nseg, st, ch == 0, false);
            }
        }
    }
    large_final_launch(A, true, nullptr, A.gpart, nullptr, st);
    return hipGetLastError() == hipSuccess ? HAWKES_OK : HAWKES_EDEVICE;
}

// one sequence of up to HK_NARROW_MAX_M nodes: segment maps and their scan, then
// one kernel per chunk
static hawkes_status run_narrow(LargeArgs& A, hipStream_t st) {
    const int32_t M = A.M;
    ZeroList Z{};
    Z.add(A.carry, (int64_t)2 * M);
    Z.add(A.seg_part, (int64_t)A.nseg * 4);
    if (A.grad && A.nchunks == 0) dense_zero(A, Z);
    large_setup_launch(A, 0, true, false, Z, st);
    for (int64_t ch = 0; ch < A.nchunks; ++ch) {
        const int64_t c0 = ch * A.CH;
        const int64_t c1 = c0 + A.CH < A.n ? c0 + A.CH : A.n;
        const int32_t nseg = (int32_t)((c1 - c0 + HK_SEG - 1) / HK_SEG);
        {
            TimedScope ts(2, st);
            hipLaunchKernelGGL(large_seg_agg, dim3(nseg), dim3(64), (size_t)2 * M * sizeof(double), st, c0, c1, M,
                               A.t, A.marks, A.beta, A.agg, A.seg_span, A.seg_dec);
        }
        {
            TimedScope ts(3, st);
            large_scan(A, nseg, nullptr, st, false);
        }
        TimedScope ts(1, st);
        const hawkes_status r = narrow_launch(A, c0, c1, nseg, ch == 0, st);
        if (r != HAWKES_OK) return r;
    }
    large_final_launch(A, true, nullptr, A.gpart, nullptr, st);
    return hipGetLastError() == hipSuccess ? HAWKES_OK : HAWKES_EDEVICE;
}

hawkes_status run_large(LargeArgs& A, hipStream_t st) {
    if (A.per_target) return run_large_pt(A, st);
    if (A.K > 1) return run_large_multi(A, st);
    if (A.narrow) return run_narrow(A, st);
    const int32_t M = A.M;
    const int64_t MM = (int64_t)M * M;
    const size_t lds_agg = (size_t)2 * M * sizeof(double);
    const size_t lds_fwd = (size_t)M * (sizeof(uint64_t) + 2 * sizeof(double));
    if (allow_lds((const void*)large_seg_agg, lds_agg) != HAWKES_OK ||
        allow_lds(Fwd<true, false, false>::kernel(M), lds_fwd) != HAWKES_OK ||
        allow_lds((const void*)large_forward<true, false, true, 1>, lds_fwd) != HAWKES_OK ||
        allow_lds(Fwd<false, true, false>::kernel(M), lds_fwd) != HAWKES_OK ||
        allow_lds(Fwd<false, false, false>::kernel(M), lds_fwd) != HAWKES_OK)
        return HAWKES_EUNSUPPORTED;
    if (A.grad && dense_allow_lds(A) != HAWKES_OK) return HAWKES_EUNSUPPORTED;
    const bool sup = A.grad && A.support;
    // support-restricted: the first term's copies (CSR order) take the place
    // of the dense partials, up to 32 of them (a power of two)
    int32_t ncopy = 1;
    while (ncopy < 32 && 2 * ncopy <= A.ER) ncopy <<= 1;
    if (sup) A.gsup = A.gpart;
    // the forward pass adds the scan's group carries itself (the scan's
    // apply pass is left out) and counts the partition (by blocks of 2^DRB
    // nodes, when the gradient needs them and they fit its LDS).  Measured
    // at c4: 6.483 -> 6.439 ms per step; also summing the chunk in the
    // forward pass's last workgroup instead of large_chunk_acc cost 0.17 ms.
    FwdExtra X;
    X.rtau = A.agg;   // free once the scan has run
    X.gcarry = A.gcarry;
    X.seg_off = A.seg_off;
    X.seg_offdec = A.seg_offdec;
    X.bs = A.DRB;
    X.nbo = A.NBO;
    X.bcnt = nullptr;
    size_t lds_fwdc = lds_fwd;   // the gradient's forward pass, with the partition counts if they fit
    if (A.grad && A.NBO <= HK_NBO_MAX) {
        const void* kf = sup ? (const void*)large_forward<true, false, true, 1>
                             : Fwd<true, false, false>::kernel(M);
        if (allow_lds(kf, lds_fwd + (size_t)A.NBO * sizeof(int32_t)) == HAWKES_OK) {
            X.bcnt = A.bo_cnt;
            lds_fwdc = lds_fwd + (size_t)A.NBO * sizeof(int32_t);
        }
    }
    A.carry_prefix = true;
    // cleared: the carried state and the segment slots' sums over the chunks
    // (one reduction after the last chunk)
    ZeroList Z{};
    Z.add(A.carry, (int64_t)2 * M);
    Z.add(A.seg_part, (int64_t)A.nseg * 4);
    if (A.grad && A.nchunks == 0) dense_zero(A, Z);
    large_setup_launch(A, 0, true, true, Z, st);
    large_index_launch(A, 0, A.csr_ptr, A.csr_cv, A.node_info, nullptr, st, sup ? A.gsup : nullptr, ncopy);
    for (int64_t ch = 0; ch < A.nchunks; ++ch) {
        const int64_t c0 = ch * A.CH;
        const int64_t c1 = c0 + A.CH < A.n ? c0 + A.CH : A.n;
        const int32_t nseg = (int32_t)((c1 - c0 + HK_SEG - 1) / HK_SEG);
        {
            TimedScope ts(2, st);
            hipLaunchKernelGGL(large_seg_agg, dim3(nseg), dim3(64), lds_agg, st, c0, c1, M, A.t, A.marks, A.beta,
                               A.agg, A.seg_span, A.seg_dec);
        }
        {
            TimedScope ts(3, st);
            large_scan(A, nseg, nullptr, st, false);
        }
        {
            TimedScope ts(1, st);
            if (sup)
                hipLaunchKernelGGL((large_forward<true, false, true, 1>), dim3(nseg), dim3(64), lds_fwdc, st, c0, c1,
                                   M, A.T, A.t, A.marks, A.mu, A.beta, A.node_info, A.csr_cv,
                                   A.carry_seg, A.seg_part, A.wchunk, (float*)nullptr, A.gsup, ncopy - 1,
                                   (double*)nullptr, (double*)nullptr, X);
            else if (A.grad)
                Fwd<true, false, false>::launch(M, nseg, lds_fwdc, st, c0, c1, M, A.T, A.t, A.marks, A.mu,
                                   A.beta, A.node_info, A.csr_cv,
                                   A.carry_seg, A.seg_part, A.wchunk, (float*)nullptr, (double*)nullptr, 0,
                                   (double*)nullptr, (double*)nullptr, X);
            else if (A.lambda_out)
                Fwd<false, true, false>::launch(M, nseg, lds_fwd, st, c0, c1, M, A.T, A.t, A.marks, A.mu,
                                   A.beta, A.node_info, A.csr_cv,
                                   A.carry_seg, A.seg_part, A.wchunk, A.lambda_out, (double*)nullptr, 0,
                                   (double*)nullptr, (double*)nullptr, X);
            else
                Fwd<false, false, false>::launch(M, nseg, lds_fwd, st, c0, c1, M, A.T, A.t, A.marks, A.mu,
                                   A.beta, A.node_info, A.csr_cv,
                                   A.carry_seg, A.seg_part, A.wchunk, (float*)nullptr, (double*)nullptr, 0,
                                   (double*)nullptr, (double*)nullptr, X);
        }
        if (A.grad) {
            {
                TimedScope tb(6, st);
                bucket_starts(A, c0, c1, nseg, A.DRB, A.bo_cnt, A.bo_off, st, X.bcnt != nullptr);
            }
            // support-restricted: only the sums per node (dL/dmu,
            // compensator) are needed
            large_dense_launch(A, c0, c1, nseg, st, ch == 0, sup);
        }
    }
    large_final_launch(A, true, nullptr, sup ? nullptr : A.gpart, A.csum, st);
    if (sup && A.g_alpha)
        hipLaunchKernelGGL(large_sup_scatter, dim3((unsigned)M), dim3(64), 0, st, M, ncopy, A.csr_ptr, A.csr_cv,
                           A.gsup, A.csum, A.g_alpha);
    return hipGetLastError() == hipSuccess ? HAWKES_OK : HAWKES_EDEVICE;
}

}  // namespace hk
