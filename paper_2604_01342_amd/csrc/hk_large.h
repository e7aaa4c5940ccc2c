// Large-M engine (M > 8, or a decay per target node): internals.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "hk_internal.h"

#ifndef HK_SEG
#define HK_SEG 1024        // events per segment (the scan's elements)
#endif
#define HK_NARROW_MAX_M 64   // nodes up to which one kernel takes the forward pass and the gradient
#define HK_F32_MIN_M 384   // nodes from which the dense gradient's U and K (and their product) are float32
#define HK_CW64 384        // widest column block with U and K in float64
#define HK_LSLOTS(BL, NCB) ((1 << (BL)) + 64 * (NCB))   // record slots of a block of events
#define HK_WIDE 60.0       // anchored-exponent limit inside one block of the dense gradient

namespace hk {

#define HK_KMAX 8          // decay kernels per problem (shared decay per kernel)

struct LargeArgs {
    int64_t n;
    int32_t M;
    int32_t K;            // decay kernels (shared decay): alpha[K][M][M], beta[K]
    int32_t per_target;   // beta[M] instead of beta[1]
    double T;
    int64_t CH;           // events per chunk
    int64_t nchunks;
    int32_t nseg;         // segments per chunk
    int32_t ER;           // event ranges of the dense kernel per chunk
    int32_t seg;          // events per segment (HK_SEG; fewer with per-target decays and few events)
    int32_t NB;           // per-target decays: node blocks of HK_PT_NB (partition and dense kernel)
    // shared decay: one kernel for few nodes (hk_narrow.hip), else hk_dense.hip
    bool narrow;
    int32_t BL;           // log2 of the events per block (6, 7 or 8; 8, 9 or 10 with several column blocks)
    int32_t DRB;          // log2 of the rows per tile (4)
    int32_t CW, NCB;      // columns per tile (a multiple of 16), column blocks
    int32_t rep;          // tile columns per node (a power of two; 1 but for few nodes)
    int32_t NSP;          // rows of spart and cpart_
    bool row64;           // rows of U and K in float64
    int32_t Mp;           // row length of urow and krow: M, padded to 64
    bool grad;
    bool support;         // dL/dalpha only at alpha's nonzeros (zero elsewhere), shared decay
    const double* t;
    const int32_t* marks;
    const float *mu, *alpha, *beta;
    // workspace (with K > 1 the per-kernel arrays below are K consecutive
    // copies: csr_*, colsum, node_info, carry, carry_seg, gpart, spart, cpart_)
    int32_t* csr_ptr;
    int2* csr_cv;         // nonzeros of alpha by row: (column, float bits of the value)
    float* colsum;
    int32_t* rcnt;        // [K][M] nonzeros per row (column, per target) of alpha
    double *rk, *dk;      // K > 1: [K][CH] per event of the chunk, R_k and D_k (alpha row . K and . J)
    double* agg;          // [nseg][2M] segment maps (K_run, J_run)
    double* seg_span;     // [nseg] time from the event before the segment to its last event
    double* seg_dec;      // [nseg] e^{-beta (span of the segment from the preceding event)}
    double* seg_off;      // [nseg] time from the event before the segment's scan group to the event before it
    double* seg_offdec;   // [nseg] e^{-beta seg_off} (shared decay)
    double* carry_seg;    // [nseg][2M] state just after the event preceding segment s
    int32_t ngr;          // scan groups per chunk
    double *gagg, *gcarry, *gspan, *gdec;   // group maps, carries, spans, decays
    int4* node_info;      // [M] (csr begin, csr end, mu, colsum)
    double* carry;        // [2M] chunk carry (K, J) just after the chunk's last event
    float* pt_flags;      // [2] per-target engine: beta_min, and (int) whether a chunk is near T
    double* seg_part;     // [nseg][2 + 2K]
    double* acc;          // [2 + 2K] call-level sums: logsum, comp, E[K], gbeta[K]
    double* ll_scratch;   // [1] log-likelihood slot when the caller wants intensities only
    bool carry_prefix;    // carry_seg holds in-group prefixes (the scan's apply pass left out)
    double *gpart, *spart, *cpart_;  // [ER][M][M]; [ER][M] (sums of w, of compensator terms or event counts)
    double* csum;         // [M] the columns' compensator sums (shared decay, gradient)
    double* gsup;         // [min(8, ER)][M*M] support-restricted first term of eq. 9 in CSR order (the
                          //   first nnz(alpha) entries of each copy; shares gpart's space)
    // dense gradient, shared decay: rows of U and K per block of events, pair
    // records per event (block order), and whether a block is wide
    double *urow, *krow;  // [CH >> BL][Mp] (and slack for a column block past the row); float32 unless row64
    uint2* prec;          // [CH] place in the block << 16 | 8 column (place 0xffff: none), e^{beta (t_j - tau_b)};
                          //   several column blocks: [CH >> BL][HK_LSLOTS], each column block's records of a
                          //   block after another, in whole groups of 64
    int32_t* plist;       // [CH >> BL][NCB + 1] first group of each column block's records (several of them)
    int32_t* wide;        // [CH >> BL]
    // per-target decays (R-form forward, reverse adjoint for the gradient)
    int32_t* csc_ptr;   // alpha by column: targets p of source q
    int2* csc_cv;       // (target, float bits of the value)
    float* wv;            // [CH] w_i = 1/lambda_i of the chunk's events
    double* pt_ck;        // [2 HK_PTCK][2M] chunk-start states (R, D): level-1 slots, then level-2 slots
    int64_t pt_ckr;       // chunks per level-1 slot
    double* ebseg;        // [nseg][M] per segment: sum_j alpha_{p,m_j} (T - t_j) e^{-beta_p (T - t_j)}
                          //   minus sum_{i: m_i = p} w_i (R_i - beta_p D_i)
    double* ebacc;        // [M] the same over the whole sequence (= -dL/dbeta_p)
    double* aggA;         // [nseg][M] reverse segment aggregates of the adjoint state
    double* rcarry_seg;   // [nseg][M] adjoint state at each segment's first event (events from there on)
    double *rgagg, *rgcarry;  // [ngr][M] reverse group aggregates and carries
    double* achunk;       // [M] adjoint state entering the current chunk from the right
    // events of the chunk partitioned by node block (64 nodes), in event order
    // (per-target decays)
    int32_t* bk_cnt;      // [NB][nseg] events per (block, segment)
    int32_t* bk_off;      // [NB][nseg + 1] start of each (block, segment) run within the block
    int32_t* bk_base;     // [NB] start of each block in the records
    uint32_t* bk_key;     // [CH] (index in chunk) << bs | mark mod 2^bs (blocks of 2^bs nodes)
    double* bk_t;         // [CH] event time
    float* bk_w;          // [CH] 1 / lambda
    float* wchunk;        // [CH] 1 / lambda of the chunk's events (shared decay)
    // the events partitioned by blocks of 2^DRB nodes: the pair kernel's own
    // events
    int32_t NBO;          // row blocks (ceil(M / 2^DRB))
    int32_t *bo_cnt, *bo_off, *bo_base;
    uint32_t* bo_key;     // [CH] (index in chunk) << DRB | mark mod 2^DRB
    float2* bo_cw;        // [CH] (beta w e^{-beta (t - tau_b)}, w)
    double* bo_e;         // [CH] 1 - e^{-beta (T - t)}
    // outputs
    double *loglik, *g_mu, *g_alpha, *g_beta;
    float* lambda_out;
};

// arrays a call clears first (large_setup)
#define HK_NZERO 6
struct ZeroList {
    double* p[HK_NZERO];
    int64_t n[HK_NZERO];
    void add(double* q, int64_t cnt) {
        for (int z = 0; z < HK_NZERO; ++z)
            if (n[z] == 0) {
                p[z] = q;
                n[z] = cnt;
                return;
            }
    }
};

// per-target decays: the shortest segment; the dense kernel's targets and
// columns per block, and the fewest events for one of its waves
#define HK_PT_SEG_MIN 256
#define HK_PT_NB 128
#define HK_PT_WAVE_EV 32
#define HK_PT_SEG_ROWS (1 << 18)   // most segments times nodes of shortened segments (15 MB of maps and states)
#define HK_SG 32           // segments per scan group
#define HK_NBO_MAX 256     // node blocks the forward pass can count for the partition

// optional parts of the shared-decay forward pass (see large_forward)
struct FwdExtra {
    double* rtau;         // [nseg][2M] scratch (the segment maps' buffer, consumed by the scan):
                          // the first M doubles of segment s hold its lazy records' times
    const double* gcarry;
    const double* seg_off;
    const double* seg_offdec;
    int32_t* bcnt;
    int32_t bs, nbo;
};
#define HK_PTCK 64         // checkpoint slots per level of the per-target gradient (at most 64^2 chunks)

// the workspace of p, carved from ws if not null; its size.  fit: if not 0 and
// the size is above it, a layout of at most that size where there is one (with
// the dense kernels tuned: longer blocks, fewer ranges, chunks half as long)
size_t large_layout(LargeArgs& A, const hawkes_problem* p, bool grad, void* ws, size_t ws_bytes, size_t fit = 0);
hawkes_status run_large(LargeArgs& A, hipStream_t st);
hawkes_status run_large_pt(LargeArgs& A, hipStream_t st);
// helpers shared by the two large-M paths (host side)
size_t lds_limit();
hawkes_status allow_lds(const void* kernel, size_t bytes, bool with_static = false);
// grants the shared-decay dense kernels their LDS
hawkes_status dense_allow_lds(const LargeArgs& A);
// colsums, index: whether column sums and nonzeros per row are wanted
void large_setup_launch(const LargeArgs& A, int trans, bool colsums, bool index, const ZeroList& Z, hipStream_t st);
void large_index_launch(const LargeArgs& A, int trans, int32_t* ptr, int2* cv, int4* node_info, float* csc_b,
                        hipStream_t st, double* gsup = nullptr, int32_t ncopy = 0);
// entries between consecutive kernels' packed rows of alpha: even (each
// kernel's array starts 16-byte aligned for the forward pass's pair loads)
// and at least one spare entry past the M^2 a dense alpha fills
inline int64_t cv_stride(int64_t MM) { return (MM + 2) & ~(int64_t)1; }
// apply = false leaves carry_seg as in-group prefixes (the forward pass and
// dense_prep then add the group carries themselves)
void large_scan(LargeArgs& A, int32_t nseg, const float* beta_pt, hipStream_t st, bool apply = true);
void large_chunk_acc_launch(int32_t nseg, int32_t width, const double* seg_part, double* acc, hipStream_t st);
void bucket_chunk(LargeArgs& A, int64_t c0, int64_t c1, int32_t nseg, const float* wchunk, int bs, hipStream_t st);
// starts of the (node block, segment) runs alone; counted: cnt already holds
// the counts (the forward pass made them)
void bucket_starts(const LargeArgs& A, int64_t c0, int64_t c1, int32_t nseg, int bs, int32_t* cnt, int32_t* off,
                   hipStream_t st, bool counted);
// first: the chunk's results replace the partials (the call's first chunk);
// sums_only: the sums per node alone (dL/dmu and the compensator), for the
// support-restricted gradient
void large_dense_launch(LargeArgs& A, int64_t c0, int64_t c1, int32_t nseg, hipStream_t st, bool first,
                        bool sums_only);

// final sums and outputs (see large_final); slots: the call-level sums are the
// segment slots' (else acc); csum: the columns' compensator sums, or null
void large_final_launch(const LargeArgs& A, bool slots, const double* ebacc, const double* gpart, double* csum,
                        hipStream_t st);

// the chunk's forward pass and gradient for up to HK_NARROW_MAX_M nodes
hawkes_status narrow_launch(const LargeArgs& A, int64_t c0, int64_t c1, int32_t nseg, bool first, hipStream_t st);

size_t seq_workspace_bytes(const hawkes_problem* p);
hawkes_status run_sequential(const hawkes_problem* p, const double* t, const int32_t* marks, const float* mu,
                             const float* alpha, const float* beta, double* loglik, double* g_mu,
                             double* g_alpha, double* g_beta, void* ws, hipStream_t st);
hawkes_status run_check_inputs(const hawkes_problem* p, const double* t, const int32_t* marks, const float* mu,
                               const float* alpha, const float* beta, int32_t* status_out, hipStream_t st);

}  // namespace hk
