// Forward pass and gradient of one sequence with 9 to 64 nodes and one shared
// decay, in one kernel: with so few nodes a group of LG = 16, 32 or 64 lanes
// holds a whole state, one node a lane, and dL/dalpha's row update is one
// instruction per event.
//
// A workgroup takes segments of HK_SEG events, two at a time (four waves
// each).  A segment's groups take 4 LG consecutive events each; their entry
// states come from the scan's carry and the groups' own maps, formed first.
// In batches of LG events a group then runs twice over its events:
//   1. R_p = sum_q alpha_pq K_q (target form: lane p) and its time-weighted
//      companion D_p: each event decays them over its gap, lane m_i hands
//      (R, D) to the event, and every lane adds its entry of the event's column
//      of alpha (LDS).  Then the events' lambda, log lambda, w = 1/lambda and
//      the partial sums, a lane an event;
//   2. K_q (lane q): decays over the gap, row m_i of the LDS tile of dL/dalpha
//      gets beta w_i K_q(t_i^-), lane m_i takes the event.
// One exponential an event, and no limit on the gaps.
// Everything is float64, and nothing is gathered per nonzero of alpha: dense
// rows cost what sparse ones do.
// Bound by instruction issue (about 30 an event of a group).  Measured against
// the passes of the large-M engine (hk_large.hip, hk_dense.hip): see
// large_layout.
#include "hk_device.h"
#include "hk_large.h"
#include "hk_stream.h"

namespace hk {

#define NA_W 8   // waves per workgroup (two segments)

__device__ __forceinline__ double recip_d(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

template <int LG, bool GRAD, bool INTENS>
__global__ __launch_bounds__(64 * NA_W) __attribute__((amdgpu_waves_per_eu(4))) void narrow_forward(int64_t c0, int64_t c1, int32_t M, double T,
                                                            const double* __restrict__ t,
                                                            const int32_t* __restrict__ marks,
                                                            const float* __restrict__ mu,
                                                            const float* __restrict__ alpha,
                                                            const float* __restrict__ beta,
                                                            const float* __restrict__ colsum,
                                                            const double* __restrict__ carry_seg,
                                                            const double* __restrict__ gcarry,
                                                            const double* __restrict__ seg_off,
                                                            const double* __restrict__ seg_offdec, int32_t nseg,
                                                            double* __restrict__ seg_part,
                                                            float* __restrict__ lambda_out,
                                                            double* __restrict__ gpart, double* __restrict__ spart,
                                                            double* __restrict__ cpart, int first) {
    constexpr int GPW = 64 / LG;          // groups per wave
    constexpr int NS = 4 * GPW;           // groups per segment
    constexpr int EPG = 4 * LG;           // events per group
    extern __shared__ double lds[];
    double* G = lds;                                              // [M][LG] (GRAD)
    float* aT = reinterpret_cast<float*>(lds + (GRAD ? M * LG : 0));   // [M][LG]: alpha by source
    __shared__ double gK[2][256], gJ[2][256];   // [group][node]: the groups' maps, then their entry states
    __shared__ double sS[GRAD ? 2 : 1][GRAD ? 256 : 1], sC[GRAD ? 2 : 1][GRAD ? 256 : 1];
    __shared__ double tg[2][NS + 1], eg[2][NS];
    __shared__ double2 slot[NA_W][64];
    __shared__ double2 stA[LG < 64 ? NA_W : 1][64];   // broadcast values of the batch
    __shared__ int32_t stM[LG < 64 ? NA_W : 1][64];
    __shared__ double red[NA_W][4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = wv >> 2, w4 = wv & 3, ht = tid & 255;
    const int l = lane & (LG - 1), g0 = lane & ~(LG - 1);
    const int grp = w4 * GPW + (lane / LG);
    const double bet = (double)beta[0];
    for (int x = tid; x < M * LG; x += 64 * NA_W) {
        const int q = x / LG, p = x % LG;
        aT[x] = p < M ? alpha[(int64_t)p * M + q] : 0.0f;
        if (GRAD) G[x] = 0.0;
    }
    if (GRAD) {
        sS[h][ht] = 0.0;
        sC[h][ht] = 0.0;
    }
    double logsum = 0.0, comp = 0.0, Esum = 0.0, gb = 0.0;
    // value v of the group's lane i, for every lane of the group
    auto bc_i = [&](int v, int i) -> int {
        if constexpr (LG == 64)
            return rl_i(v, i);
        else
            return stM[wv][g0 + i];
    };
    for (int32_t s2 = blockIdx.x * 2; s2 < nseg; s2 += (int32_t)gridDim.x * 2) {
        const int32_t s = s2 + h;
        const bool live = s < nseg;
        const int64_t a = c0 + (int64_t)(live ? s : 0) * HK_SEG;
        const int64_t b = live ? (a + HK_SEG < c1 ? a + HK_SEG : c1) : a;
        __syncthreads();   // the last segments' entry states are read
        gK[h][ht] = 0.0;
        gJ[h][ht] = 0.0;
        if (ht <= NS) {
            // time of the event before group ht (NS: the last event)
            const int64_t e = a + (int64_t)ht * EPG < b ? a + (int64_t)ht * EPG : b;
            tg[h][ht] = t[e > 0 ? e - 1 : 0];
        }
        __syncthreads();
        if (ht < NS) eg[h][ht] = exp_f64(-bet * (tg[h][ht + 1] - tg[h][ht]));
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = 256 * w4 + 64 * u + lane;
            const int64_t i = a + e;
            if (i < b) {
                const int ge = e / EPG;
                const double d = tg[h][ge + 1] - t[i];
                const double x = exp_f64(-bet * d);
                const int m = clamp_mark(marks[i], M);
                atomicAdd(&gK[h][ge * LG + m], x);
                if (GRAD) atomicAdd(&gJ[h][ge * LG + m], d * x);
            }
        }
        __syncthreads();
        if (live && ht < M) {
            // chain of the groups' maps from the segment's carry
            const double* cs = carry_seg + (int64_t)s * 2 * M;
            const double* gc = gcarry + (int64_t)(s / HK_SG) * 2 * M;
            const double Dg = seg_off[s], exg = seg_offdec[s];
            const double Kc = gc[ht];
            double K = __builtin_fma(exg, Kc, cs[ht]);
            double J = __builtin_fma(exg, __builtin_fma(Dg, Kc, gc[M + ht]), cs[M + ht]);
            for (int g = 0; g < NS; ++g) {
                const double k = gK[h][g * LG + ht], j = gJ[h][g * LG + ht];
                gK[h][g * LG + ht] = K;
                gJ[h][g * LG + ht] = J;
                const double ex = eg[h][g], D = tg[h][g + 1] - tg[h][g];
                J = __builtin_fma(ex, __builtin_fma(D, K, J), j);
                K = __builtin_fma(ex, K, k);
            }
        }
        __syncthreads();
        if (!live) continue;
        const int64_t ga = a + (int64_t)grp * EPG;   // the group's first event
        // this lane's node: K_l, and R_l, D_l from the group's entry state
        double K0 = gK[h][grp * LG + l], R0 = 0.0, D0 = 0.0;
#pragma unroll 4
        for (int q = 0; q < M; ++q) {
            const double av = (double)aT[q * LG + l];
            R0 = __builtin_fma(av, gK[h][grp * LG + q], R0);
            if (GRAD) D0 = __builtin_fma(av, gJ[h][grp * LG + q], D0);
        }
        if (l >= M) K0 = 0.0;
        double ta = tg[h][grp];
        double tn;
        int mn;
        auto ld = [&](int bt) {
            const int64_t i = ga + bt * LG + l;
            const int64_t ic = i < b ? i : b - 1;
            tn = t[ic];
            mn = clamp_mark(marks[ic], M);
        };
        ld(0);
        for (int bt = 0; bt < 4; ++bt) {
            // pass 1 (a chain) before other waves' pass 2 (LDS adds): 92 / 88
            // us at M = 50, 1e6 events
            __builtin_amdgcn_s_setprio(2);
            const int64_t i = ga + bt * LG + l;
            const bool valid = i < b;
            if (__ballot(valid) == 0) break;
            const double ti = valid ? tn : ta;
            const int mi = valid ? mn : 0;
            if (bt < 3) ld(bt + 1);
            // time from the event before, and the decay over it (past the
            // sequence's end: none; nothing follows there)
            double tp = __shfl_up(ti, 1, 64);
            tp = l == 0 ? ta : tp;
            const double F = valid ? ti - tp : 0.0, d = exp_f64(-bet * F);
            // pass 1: four events at a time, their broadcasts and columns of
            // alpha read before the first is taken
            if (LG < 64) {
                stA[wv][lane] = make_double2(d, F);
                stM[wv][lane] = mi;
                lds_wait();
            }
            for (int k0 = 0; k0 < LG; k0 += 4) {
                int m[4];
                double dk[4], Fk[4];
                float av[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    m[j] = bc_i(mi, k0 + j);
                    if constexpr (LG == 64) {
                        dk[j] = rl_d(d, k0 + j);
                        Fk[j] = GRAD ? rl_d(F, k0 + j) : 0.0;
                    } else {
                        const double2 x = stA[wv][g0 + k0 + j];
                        dk[j] = x.x;
                        Fk[j] = x.y;
                    }
                    av[j] = aT[m[j] * LG + l];
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (GRAD) D0 = dk[j] * __builtin_fma(Fk[j], R0, D0);
                    R0 = dk[j] * R0;
                    if (l == m[j]) slot[wv][g0 + k0 + j] = make_double2(R0, D0);
                    R0 += (double)av[j];
                }
            }
            lds_wait();
            double c = 0.0;
            {
                const double2 sv = slot[wv][lane];
                const double R = sv.x, D = sv.y;
                const double x = bet * (T - ti);
                const double ex = exp_f64(-x);
                const double em1 = __ballot(valid && x < 0.5) == 0 ? 1.0 - ex : -expm1(-x);
                if (valid) {
                    const double lam = __builtin_fma(bet, R, (double)mu[mi]);
                    const double cm = (double)colsum[mi];
                    if (INTENS) lambda_out[i] = (float)lam;
                    logsum += log(lam);
                    comp += cm * em1;
                    if (GRAD) {
                        const double w = recip_d(lam);
                        Esum += cm * (T - ti) * ex;
                        gb += w * (R - bet * D);
                        c = bet * w;
                        atomicAdd(&sS[h][grp * LG + mi], w);
                        atomicAdd(&sC[h][grp * LG + mi], em1);
                    }
                }
            }
            if (GRAD) {
                __builtin_amdgcn_s_setprio(0);
                // pass 2
                if (LG < 64) {
                    stA[wv][lane] = make_double2(d, c);
                    lds_wait();
                }
                for (int k0 = 0; k0 < LG; k0 += 4) {
                    int m[4];
                    double dk[4], ck[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        m[j] = bc_i(mi, k0 + j);
                        if constexpr (LG == 64) {
                            dk[j] = rl_d(d, k0 + j);
                            ck[j] = rl_d(c, k0 + j);
                        } else {
                            const double2 x = stA[wv][g0 + k0 + j];
                            dk[j] = x.x;
                            ck[j] = x.y;
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        K0 *= dk[j];
                        atomicAdd(&G[m[j] * LG + l], ck[j] * K0);
                        K0 += l == m[j] ? 1.0 : 0.0;
                    }
                }
            }
            ta = __shfl(ti, g0 + LG - 1, 64);
        }
    }
    __syncthreads();
    // the workgroup's partial sums, in a fixed order
    for (int off = 32; off > 0; off >>= 1) {
        logsum += __shfl_down(logsum, off, 64);
        comp += __shfl_down(comp, off, 64);
        Esum += __shfl_down(Esum, off, 64);
        gb += __shfl_down(gb, off, 64);
    }
    if (lane == 0) {
        red[wv][0] = logsum;
        red[wv][1] = comp;
        red[wv][2] = Esum;
        red[wv][3] = gb;
    }
    __syncthreads();
    if (tid < 4) {
        double v = 0.0;
        for (int k = 0; k < NA_W; ++k) v += red[k][tid];
        seg_part[(int64_t)blockIdx.x * 4 + tid] += v;
    }
    if (!GRAD) return;
    if (tid < M) {
        double sv = 0.0, cv = 0.0;
        for (int k = 0; k < 2; ++k)
            for (int g = 0; g < NS; ++g) {
                sv += sS[k][g * LG + tid];
                cv += sC[k][g * LG + tid];
            }
        const int64_t o = (int64_t)blockIdx.x * M + tid;
        spart[o] = first ? sv : spart[o] + sv;
        cpart[o] = first ? cv : cpart[o] + cv;
    }
    double* gp = gpart + (int64_t)blockIdx.x * M * M;
    for (int x = tid; x < M * M; x += 64 * NA_W) {
        const double v = G[(x / M) * LG + x % M];
        gp[x] = first ? v : gp[x] + v;
    }
}

// ------------------------------------------------------------------ host
static size_t narrow_lds(const LargeArgs& A, int LG) {
    return (size_t)A.M * LG * (sizeof(float) + (A.grad ? sizeof(double) : 0));
}

template <int LG>
static hawkes_status narrow_launch_t(const LargeArgs& A, int64_t c0, int64_t c1, int32_t nseg, bool first,
                                     hipStream_t st) {
    auto go = [&](auto* kern) {
        const size_t bytes = narrow_lds(A, LG);
        if (allow_lds((const void*)kern, bytes, true) != HAWKES_OK) return HAWKES_EUNSUPPORTED;
        hipLaunchKernelGGL(kern, dim3((unsigned)A.ER), dim3(64 * NA_W), bytes, st, c0, c1, A.M, A.T, A.t, A.marks,
                           A.mu, A.alpha, A.beta, A.colsum, A.carry_seg, A.gcarry, A.seg_off, A.seg_offdec, nseg,
                           A.seg_part, A.lambda_out, A.gpart, A.spart, A.cpart_, first ? 1 : 0);
        return HAWKES_OK;
    };
    if (A.grad) return go(narrow_forward<LG, true, false>);
    if (A.lambda_out) return go(narrow_forward<LG, false, true>);
    return go(narrow_forward<LG, false, false>);
}

hawkes_status narrow_launch(const LargeArgs& A, int64_t c0, int64_t c1, int32_t nseg, bool first, hipStream_t st) {
    if (A.M <= 16) return narrow_launch_t<16>(A, c0, c1, nseg, first, st);
    if (A.M <= 32) return narrow_launch_t<32>(A, c0, c1, nseg, first, st);
    return narrow_launch_t<64>(A, c0, c1, nseg, first, st);
}

}  // namespace hk
