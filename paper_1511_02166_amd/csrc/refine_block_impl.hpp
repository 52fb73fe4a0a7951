// refine_block_impl.hpp -- one workgroup refines one airfoil's FP32 solutions
// against the FP64 system (device functions only).
//
// Iterative refinement of X with the FP64 system in A64 and the FP32 factors
// in A32.  One sweep: r = b - A x in FP64; for each right-hand side not yet
// converged: stop if r is at the FP64 backward-error floor, ||r||_inf <=
// sqrt(n) eps ||A||_inf ||x||_inf (no further sweep can improve x); otherwise
// d = U^{-1} L^{-1} P r in FP32, x += d, and stop by the rule of
// refined_enough.
//
// A sweep is bound by reading A64 and the factors, so up to KG right-hand
// sides share one read of each.  Both the residual and the off-diagonal part
// of the triangular solves run on the matrix cores as D = X^T A^T (source A a
// 16 (right-hand sides) x 4 slice of the solutions, source B four columns of
// 16 consecutive rows): one load of the matrix feeds all the right-hand sides
// and costs one instruction.  (With a row per thread on the vector ALUs, four
// right-hand sides per pass were the most that fitted in registers: 256
// systems of order 1025 with eight right-hand sides took 4.7 ms, now 1.4.)
#pragma once

#include "lu_wave_impl.hpp"
#include "panel_internal.hpp"
#include "wave.hpp"

namespace panel {
namespace {
namespace rfb {

using wv::TileMap;
using wv::mfma_t;
using wv::opaque_s;

constexpr int SB = 64;     // rows per diagonal block in the triangular solves

// Maximum over each row of 16 lanes, in all its lanes.
__device__ __forceinline__ double row16_max(double v) {
    v = fmax(v, dpp_d<0xB1>(v));    // quad_perm [1,0,3,2]
    v = fmax(v, dpp_d<0x4E>(v));    // quad_perm [2,3,0,1]
    v = fmax(v, dpp_d<0x141>(v));   // row_half_mirror
    return fmax(v, dpp_d<0x140>(v));   // row_mirror
}

// KG: right-hand sides per pass (4 or 8); NM: largest order.
template <int TB, int KG, int NM> struct WgRefLds {
    static constexpr int W = TB / 64;
    double sx[NM * KG];           // current solutions, [row][right-hand side]
    alignas(16) float sd[NM * KG];   // residuals by pivot position, then the corrections
    union {
        float sblk[SB * SB];                     // a diagonal block of the factors
        double part[W][2][64][KG / 4];           // partial sums of a residual tile
    } u;
    double rpart[W][32];          // partial row sums of |A|
    double red[KG][W];
    unsigned short perm[NM], pinv[NM];
};

// Solve the diagonal block [rb, rb + w) for all right-hand sides, one or two
// per wavefront side by side (lane = row); LOWER: unit lower, else upper.
template <bool LOWER, int TB, int KG, typename Lds>
__device__ __forceinline__ void diag_solve(int rb, int w, Lds &S) {
    constexpr int W = TB / 64, NR = (KG + W - 1) / W;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wave >= KG) return;
    const float *sblk = S.u.sblk;
    float y[NR];
#pragma unroll
    for (int m = 0; m < NR; ++m) y[m] = lane < w ? S.sd[(rb + lane) * KG + wave + W * m] : 0.0f;
    const float dinv = LOWER ? 1.0f : lane < w ? 1.0f / sblk[lane * SB + lane] : 0.0f;
#pragma unroll 1
    for (int jb = 0; jb < SB; jb += 8) {
        const int j0 = LOWER ? jb : SB - 8 - jb;
        if (j0 >= w) continue;
        float a[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] = sblk[(j0 + j) * SB + lane];
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const int j = LOWER ? jj : 7 - jj;
            if (j0 + j < w) {
#pragma unroll
                for (int m = 0; m < NR; ++m) {
                    if (!LOWER && lane == j0 + j) y[m] *= dinv;
                    const float xj = readlane_t(y[m], j0 + j);
                    if (LOWER ? lane > j0 + j : lane < j0 + j) y[m] -= a[j] * xj;
                }
            }
        }
    }
#pragma unroll
    for (int m = 0; m < NR; ++m)
        if (lane < w) S.sd[(rb + lane) * KG + wave + W * m] = y[m];
}

// L y = y (unit lower) or U y = y for the KG vectors in S.sd.
template <bool LOWER, int TB, int KG, typename Lds>
__device__ __forceinline__ void tri_solve(const float *F, int ld, int n, Lds &S) {
    constexpr int W = TB / 64, E = SB * SB / TB;
    typedef TileMap<float>::acc acc_t;
    typedef float f4_t __attribute__((ext_vector_type(4)));
    ld = opaque_s(ld);
    const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, k4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (n + SB - 1) / SB;
    float db[E];   // the next diagonal block on its way to LDS
    auto load_diag = [&](int blk) {
        const int rb = blk * SB;
        const int r = min(rb + lane, n - 1);
#pragma unroll
        for (int e = 0; e < E; ++e) db[e] = F[(size_t)min(rb + wave + W * e, n - 1) * ld + r];
    };
    load_diag(LOWER ? 0 : nblk - 1);
#pragma unroll 1
    for (int bb = 0; bb < nblk; ++bb) {
        const int blk = LOWER ? bb : nblk - 1 - bb;
        const int rb = blk * SB, w = min(SB, n - rb);
#pragma unroll
        for (int e = 0; e < E; ++e) S.u.sblk[(wave + W * e) * SB + lane] = db[e];
        load_diag(LOWER ? min(blk + 1, nblk - 1) : max(blk - 1, 0));
        // rows that take this block's contribution, 32 per wavefront at a time
        const int r0 = LOWER ? rb + SB : 0, r1 = LOWER ? n : rb;
        float lf[2][16];
        auto load_f = [&](int r) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int rr = max(min(r + 16 * t + i16, r1 - 1), 0);
#pragma unroll
                for (int s = 0; s < 16; ++s) lf[t][s] = F[(size_t)(rb + min(4 * s + k4, w - 1)) * ld + rr];
            }
        };
        if (r0 + 32 * wave < r1) load_f(r0 + 32 * wave);
        lds_barrier();
        diag_solve<LOWER, TB, KG>(rb, w, S);
        lds_barrier();
        float xa[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int k = 4 * s + k4;
            xa[s] = k < w ? -S.sd[(rb + min(k, w - 1)) * KG + (i16 & (KG - 1))] : 0.0f;
        }
#pragma unroll 1
        for (int r = r0 + 32 * wave; r < r1; r += 32 * W) {
            acc_t a0[2], a1[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) a0[t][e] = a1[t][e] = 0.0f;
#pragma unroll
            for (int s = 0; s < 16; s += 2)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    a0[t] = mfma_t(xa[s], lf[t][s], a0[t]);
                    a1[t] = mfma_t(xa[s + 1], lf[t][s + 1], a1[t]);
                }
            if (r + 32 * W < r1) load_f(r + 32 * W);
            // right-hand sides 4 k4 .. 4 k4 + 3 of row i16
            if (4 * k4 < KG) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int rr = r + 16 * t + i16;
                    if (rr < r1) {
                        f4_t *c = reinterpret_cast<f4_t *>(&S.sd[rr * KG + 4 * k4]);
                        f4_t v = *c;
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += a0[t][e] + a1[t][e];
                        *c = v;
                    }
                }
            }
        }
        lds_barrier();
    }
}

// Partial residual of 32 rows over the columns [kb, ke): acc[t][e] -= sum_k
// A[row][k] x[k][rhs] (rhs = k4 + 4 e, row = r0 + 16 t + i16), and with NORM
// the sums of |A| over this lane's columns.
template <int KG, bool NORM, typename Lds>
__device__ __forceinline__ void resid_tile(const double *A, int ld, int n, int r0, int kb, int ke,
                                           TileMap<double>::acc (&acc)[2], double (&ra)[2], Lds &S) {
    constexpr int KS = 8;   // k-steps (of four columns) per round trip
    const int lane = threadIdx.x & 63, i16 = lane & 15, k4 = lane >> 4;
    const double *ap[2] = {A + min(r0 + i16, n - 1), A + min(r0 + 16 + i16, n - 1)};
    double a[2][KS];
    auto load_a = [&](int k0) {
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const size_t c = (size_t)min(k0 + 4 * s + k4, n - 1) * ld;
#pragma unroll
            for (int t = 0; t < 2; ++t) a[t][s] = ap[t][c];
        }
    };
    load_a(kb);
#pragma unroll 1
    for (int k0 = kb; k0 < ke; k0 += 4 * KS) {
        double b[2][KS];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int s = 0; s < KS; ++s) b[t][s] = a[t][s];
        load_a(k0 + 4 * KS);
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k = k0 + 4 * s + k4;
            const double x = k < ke ? -S.sx[min(k, n - 1) * KG + (i16 & (KG - 1))] : 0.0;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                acc[t] = mfma_t(x, b[t][s], acc[t]);
                if (NORM) ra[t] += k < ke ? fabs(b[t][s]) : 0.0;
            }
        }
    }
}

// Residuals of the group's solutions: to S.sd by pivot position, their sizes
// (of right-hand side tid % KG) to m, and with NORM ||A||_inf to anrm.
template <int TB, int KG, bool NORM, typename Lds>
__device__ __forceinline__ void residual(const double *A, int ld, int n, int k0, int kn, double &m, double &anrm,
                                         Lds &S) {
    constexpr int W = TB / 64;
    typedef TileMap<double>::acc acc_t;
    ld = opaque_s(ld);
    const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, k4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = (n + 31) / 32, full = nt / W * W;
    double rmax[KG / 4], rowmax = 0.0;
#pragma unroll
    for (int e = 0; e < KG / 4; ++e) rmax[e] = 0.0;
    auto start = [&](acc_t (&acc)[2], int r0, bool with_b) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[t][e] = with_b && e < KG / 4
                                ? A[(size_t)(n + k0 + min(k4 + 4 * e, kn - 1)) * ld + min(r0 + 16 * t + i16, n - 1)]
                                : 0.0;
    };
    auto finish = [&](int row, int e, double r) {
        S.sd[S.pinv[row] * KG + k4 + 4 * e] = (float)r;
        rmax[e] = fmax(rmax[e], fabs(r));
    };
    for (int tile = wave; tile < full; tile += W) {
        const int r0 = 32 * tile;
        acc_t acc[2];
        double ra[2] = {0.0, 0.0};
        start(acc, r0, true);
        resid_tile<KG, NORM>(A, ld, n, r0, 0, n, acc, ra, S);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int row = r0 + 16 * t + i16;
            if (row < n) {
#pragma unroll
                for (int e = 0; e < KG / 4; ++e) finish(row, e, acc[t][e]);
            }
            if (NORM) {
                ra[t] += __shfl_xor(ra[t], 16);
                ra[t] += __shfl_xor(ra[t], 32);
                if (row < n) rowmax = fmax(rowmax, ra[t]);
            }
        }
    }
    // the tiles left over are split by columns over the wavefronts (a round
    // of its own for a few rows would leave most of the workgroup idle)
    const int kc = ((n + W - 1) / W + 3) & ~3;
    for (int tile = full; tile < nt; ++tile) {
        const int r0 = 32 * tile;
        acc_t acc[2];
        double ra[2] = {0.0, 0.0};
        start(acc, r0, wave == 0);
        const int kb = min(kc * wave, n), ke = min(kb + kc, n);
        if (kb < ke) resid_tile<KG, NORM>(A, ld, n, r0, kb, ke, acc, ra, S);
        lds_barrier();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int e = 0; e < KG / 4; ++e) S.u.part[wave][t][lane][e] = acc[t][e];
            if (NORM) {
                ra[t] += __shfl_xor(ra[t], 16);
                ra[t] += __shfl_xor(ra[t], 32);
                if (k4 == 0) S.rpart[wave][16 * t + i16] = ra[t];
            }
        }
        lds_barrier();
        if (wave < 2) {   // wavefront t sums row tile t
            const int row = r0 + 16 * wave + i16;
            if (row < n) {
#pragma unroll
                for (int e = 0; e < KG / 4; ++e) {
                    double r = S.u.part[0][wave][lane][e];
                    for (int w = 1; w < W; ++w) r += S.u.part[w][wave][lane][e];
                    finish(row, e, r);
                }
                if (NORM) {
                    double r = 0.0;
                    for (int w = 0; w < W; ++w) r += S.rpart[w][16 * wave + i16];
                    rowmax = fmax(rowmax, r);
                }
            }
        }
    }
    lds_barrier();
#pragma unroll
    for (int e = 0; e < KG / 4; ++e) {
        const double r = row16_max(rmax[e]);
        if (i16 == 0) S.red[k4 + 4 * e][wave] = r;
    }
    if (NORM) {
        rowmax = wave_max(rowmax);
        if (lane == 0) S.rpart[wave][0] = rowmax;
    }
    lds_barrier();
    m = S.red[tid % KG][0];
    for (int w = 1; w < W; ++w) m = fmax(m, S.red[tid % KG][w]);
    if (NORM) {
        anrm = S.rpart[0][0];
        for (int w = 1; w < W; ++w) anrm = fmax(anrm, S.rpart[w][0]);
    }
    lds_barrier();
}

// Maximum over the threads of the same right-hand side (tid % KG).
template <int TB, int KG, typename Lds>
__device__ __forceinline__ double group_max(double x, Lds &S) {
    constexpr int W = TB / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int off = KG; off < 64; off <<= 1) x = fmax(x, __shfl_xor(x, off));
    if (lane < KG) S.red[lane][wave] = x;
    lds_barrier();
    x = S.red[tid % KG][0];
    for (int w = 1; w < W; ++w) x = fmax(x, S.red[tid % KG][w]);
    lds_barrier();
    return x;
}

template <int TB, int KG, int NM>
__device__ __forceinline__ void wg_refine(const WsView &v, int b, int32_t *__restrict__ info, double tol,
                                          int max_iter, WgRefLds<TB, KG, NM> &S) {
    const AirfoilMeta mt = v.meta[b];
    const int n = mt.n1, ld = mt.ld;
    const int tid = threadIdx.x;
    double *X = v.x + mt.x_off;
    const int before = info[b];   // (read by all before it is written below)
    if (before != 0 || n > NM) {
        // not factored, or a system too large for this instance (-3: the
        // workspace's airfoil order does not match the plan)
        const int code = before != 0 ? before : -3;
        if (before == 0)
            for (int i = tid; i < n * mt.K; i += TB) X[i] = __builtin_nan("");
        __syncthreads();
        if (tid == 0) {
            v.iters[b] = 0;
            info[b] = code;
            v.flag[b] = code;
        }
        return;
    }
    const double *A = v.a64 + mt.a_off;
    const float *LU = v.a32 + mt.a_off;
    perm_of_pivots(v.piv + mt.piv_off, n, TB, S.perm);
    for (int i = tid; i < n; i += TB) S.pinv[S.perm[i]] = (unsigned short)i;
    const double floor_c = sqrt((double)n) * 2.220446049250313e-16;
    double anrm = -1.0;   // ||A||_inf, found during the first residual
    int worst = 0;
    bool failed = max_iter == 0;
    const int rhs = tid % KG;   // this thread's right-hand side in elementwise passes
    for (int k0 = 0; k0 < mt.K; k0 += KG) {
        const int kn = min(KG, mt.K - k0);
        // (right-hand sides past the last repeat it and are not written back)
        double x0 = 0.0;
        for (int i = tid / KG; i < n; i += TB / KG) {
            const double x = X[(size_t)(k0 + min(rhs, kn - 1)) * n + i];
            S.sx[i * KG + rhs] = x;
            x0 = fmax(x0, fabs(x));
        }
        __syncthreads();
        // state of this thread's right-hand side; `conv` (bit k: right-hand
        // side k is done) is the same in every thread
        double xn = group_max<TB, KG>(x0, S), dprev = -1.0;
        int sweeps = 0;
        bool mine = rhs >= kn;
        constexpr unsigned ALL = (1u << KG) - 1u;
        unsigned conv = (unsigned)__ballot(mine) & ALL;
        for (int it = 0; it < max_iter && conv != ALL; ++it) {
            double m;
            if (anrm < 0.0)
                residual<TB, KG, true>(A, ld, n, k0, kn, m, anrm, S);
            else
                residual<TB, KG, false>(A, ld, n, k0, kn, m, anrm, S);
            // a right-hand side whose residual is at the FP64 backward-error
            // floor is done; the others take a correction
            mine = mine || m <= floor_c * anrm * xn;
            conv = (unsigned)__ballot(mine) & ALL;
            if (conv == ALL) break;
            tri_solve<true, TB, KG>(LU, ld, n, S);
            tri_solve<false, TB, KG>(LU, ld, n, S);
            double d0 = 0.0, d1 = 0.0;
            if (!mine) {
                for (int i = tid / KG; i < n; i += TB / KG) {
                    const double dd = (double)S.sd[i * KG + rhs];
                    const double x1 = S.sx[i * KG + rhs] + dd;
                    S.sx[i * KG + rhs] = x1;
                    d0 = fmax(d0, fabs(dd));
                    d1 = fmax(d1, fabs(x1));
                }
            }
            d0 = group_max<TB, KG>(d0, S);
            d1 = group_max<TB, KG>(d1, S);
            if (!mine) {
                ++sweeps;
                xn = d1;
                mine = wv::refined_enough(d0, dprev, xn, tol);
                dprev = d0;
            }
            conv = (unsigned)__ballot(mine) & ALL;
        }
        if (conv != ALL) failed = true;
        worst = max(worst, sweeps);
        if (rhs < kn)
            for (int i = tid / KG; i < n; i += TB / KG) X[(size_t)(k0 + rhs) * n + i] = S.sx[i * KG + rhs];
        __syncthreads();
    }
    for (int off = 1; off < KG; off <<= 1) worst = max(worst, __shfl_xor(worst, off));
    if (tid == 0) {
        v.iters[b] = worst;
        if (failed) info[b] = -2;
        v.flag[b] = info[b];
    }
}

}  // namespace rfb
}  // namespace
}  // namespace panel
