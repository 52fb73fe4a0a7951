// adjoint_impl.hpp -- the transposed solve shared by the adjoint kernels: one
// workgroup per airfoil, any order up to NM (device functions only).
#pragma once

#include "fastmath.hpp"
#include "panel_internal.hpp"
#include "wave.hpp"

namespace panel {
namespace {
namespace adj {

constexpr int SB = 64;      // unknowns per diagonal block
constexpr int SBP = SB + 1; // its row stride in LDS

template <typename T> __device__ inline const T *factors(const WsView &v, const AirfoilMeta &mt);
template <> __device__ inline const double *factors<double>(const WsView &v, const AirfoilMeta &mt) {
    return v.a64 + mt.a_off;
}
template <> __device__ inline const float *factors<float>(const WsView &v, const AirfoilMeta &mt) {
    return v.a32 + mt.a_off;
}

// sum over 64 lanes, in T
__device__ __forceinline__ double lane_sum(double v) { return wave_sum(v); }
__device__ __forceinline__ float lane_sum(float v) {
    v += dpp_f<0xB1>(v);
    v += dpp_f<0x4E>(v);
    v += dpp_f<0x141>(v);
    v += dpp_f<0x140>(v);
    return (readlane_f(v, 0) + readlane_f(v, 16)) + (readlane_f(v, 32) + readlane_f(v, 48));
}

// LDS of the transposed solve.
template <typename T, int TB> struct SolveLds {
    T sblk[SB * SBP];
    T part[SB];
};

// sum_j M[j, c] y[j] over the rows [j0, j1) of column c, for up to CN columns
// c0, c0 + step, .. < c1 of one wavefront side by side: lanes along the
// column, so every load is a run of 64 entries.
template <typename T, int CN>
__device__ __forceinline__ void column_dots(const T *M, int ld, int c0, int step, int c1, int j0, int j1, const T *y,
                                            T (&s)[CN]) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < CN; ++k) s[k] = T(0);
    for (int j = j0; j < j1; j += 128) {
        T a[2][CN];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < CN; ++k)
                a[h][k] = M[(size_t)min(c0 + k * step, c1 - 1) * ld + min(j + 64 * h + lane, j1 - 1)];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = j + 64 * h + lane;
            const T yj = r < j1 ? y[min(r, j1 - 1)] : T(0);
#pragma unroll
            for (int k = 0; k < CN; ++k) s[k] += a[h][k] * yj;
        }
    }
#pragma unroll
    for (int k = 0; k < CN; ++k) s[k] = lane_sum(s[k]);
}

// Solve U^T z = y (UPPER) or L^T z = y (unit lower) in place, y in LDS.  Row i
// of the transposed factor is column i, contiguous in memory.
template <bool UPPER, typename T, int TB>
__device__ __forceinline__ void trsv_t(const T *F, int ld, int n, T *y, SolveLds<T, TB> &S) {
    constexpr int W = TB / 64, CN = 4, E = SB * SB / TB;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nblk = (n + SB - 1) / SB;
    for (int bb = 0; bb < nblk; ++bb) {
        const int blk = UPPER ? bb : nblk - 1 - bb;
        const int rb = blk * SB, w = min(SB, n - rb), re = rb + w;
        // the diagonal block (its other triangle is read too and never used)
        T d[E];
#pragma unroll
        for (int e = 0; e < E; ++e) d[e] = F[(size_t)min(rb + wave + W * e, n - 1) * ld + min(rb + lane, n - 1)];
        // the solved unknowns' share of the block's rows
        const int j0 = UPPER ? 0 : re, j1 = UPPER ? rb : n;
        for (int c = wave; c < w; c += CN * W) {
            T s[CN];
            column_dots<T, CN>(F, ld, rb + c, W, re, j0, j1, y, s);
#pragma unroll
            for (int k = 0; k < CN; ++k)
                if (lane == 0 && c + k * W < w) S.part[c + k * W] = s[k];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) S.sblk[(wave + W * e) * SBP + lane] = d[e];
        __syncthreads();
        if (wave == 0) {
            // lane i: unknown rb + i; its row of the transposed block is
            // column i of the block
            T yi = T(0), dinv = T(1);
            if (lane < w) {
                yi = y[rb + lane] - S.part[lane];
                if (UPPER) dinv = T(1) / S.sblk[lane * SBP + lane];
            }
            const T *row = S.sblk + lane * SBP;
#pragma unroll 1
            for (int jb = 0; jb < SB; jb += 8) {
                const int b0 = UPPER ? jb : SB - 8 - jb;
                if (b0 >= w) continue;
                T a[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) a[j] = row[b0 + j];
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) {
                    const int j = UPPER ? jj : 7 - jj;
                    if (b0 + j < w) {
                        if (UPPER && lane == b0 + j) yi *= dinv;
                        const T zj = readlane_t(yi, b0 + j);
                        if (UPPER ? lane > b0 + j : lane < b0 + j) yi -= a[j] * zj;
                    }
                }
            }
            if (lane < w) y[rb + lane] = yi;
        }
        __syncthreads();
    }
}

// out[perm[i]] = (P^T-ordered) solution of (P^T L U)^T out = y; y clobbered.
template <typename T, int TB, typename O>
__device__ __forceinline__ void solve_t(const T *LU, int ld, int n, const unsigned short *perm, T *y, O *out,
                                        SolveLds<T, TB> &S) {
    trsv_t<true, T, TB>(LU, ld, n, y, S);
    trsv_t<false, T, TB>(LU, ld, n, y, S);
    for (int i = threadIdx.x; i < n; i += TB) out[perm[i]] = O(y[i]);
    __syncthreads();
}

// Workgroup-wide maxima of three values.
template <int TB>
__device__ __forceinline__ void block_max3(double &a, double &b, double &c, double (*red)[TB / 64]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    a = wave_max(a);
    b = wave_max(b);
    c = wave_max(c);
    if (lane == 0) {
        red[0][wave] = a;
        red[1][wave] = b;
        red[2][wave] = c;
    }
    __syncthreads();
    a = red[0][0];
    b = red[1][0];
    c = red[2][0];
    for (int w = 1; w < TB / 64; ++w) {
        a = fmax(a, red[0][w]);
        b = fmax(b, red[1][w]);
        c = fmax(c, red[2][w]);
    }
    __syncthreads();
}

// Vectors of the FP32 refinement of lambda (nothing for FP64 factors).
template <typename T, int NM> struct LambdaLds {};
template <int NM> struct LambdaLds<float, NM> {
    float y[NM];
    double wv[NM];
};

// lambda = M^{-T} w for airfoil mt: w in tmp on entry (clobbered), lambda in
// lam on exit.  FP64 factors: one transposed solve.  FP32 factors: lambda from
// U^T / L^T in FP32, then FP64 refinement of the transposed system against
// the FP64 matrix kept in A64.  Returns false when the refinement ran out of
// sweeps.
template <typename T, int TB, int NM>
__device__ __forceinline__ bool solve_lambda(const WsView &v, const AirfoilMeta &mt, const unsigned short *perm,
                                             double *lam, double *tmp, SolveLds<T, TB> &S, LambdaLds<T, NM> &Lx,
                                             double (*red)[TB / 64]) {
    const int n = mt.n1, ld = mt.ld;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const T *LU = factors<T>(v, mt);
    if constexpr (sizeof(T) == 8) {
        solve_t<double, TB, double>(LU, ld, n, perm, tmp, lam, S);
        return true;
    } else {
        constexpr int W = TB / 64, CN = 4;
        const double *A = v.a64 + mt.a_off;
        for (int i = tid; i < n; i += TB) {
            Lx.wv[i] = tmp[i];
            Lx.y[i] = (float)tmp[i];
        }
        __syncthreads();
        solve_t<float, TB, double>(LU, ld, n, perm, Lx.y, lam, S);
        const double floor_c = sqrt((double)n) * 2.220446049250313e-16;
        double anrm = -1.0;
        for (int it = 0; it < 10; ++it) {
            // r = w - A^T lambda: a wavefront per column of A
            double rmax = 0.0, lmax = 0.0, cmax = 0.0;
            for (int i = tid; i < n; i += TB) lmax = fmax(lmax, fabs(lam[i]));
            for (int c = wave; c < n; c += CN * W) {
                double s[CN], ca[CN];
#pragma unroll
                for (int k = 0; k < CN; ++k) s[k] = ca[k] = 0.0;
                for (int j = 0; j < n; j += 128) {
                    double a[2][CN];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int k = 0; k < CN; ++k)
                            a[h][k] = A[(size_t)min(c + k * W, n - 1) * ld + min(j + 64 * h + lane, n - 1)];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int r = j + 64 * h + lane;
                        const bool in = r < n;
                        const double l = in ? lam[min(r, n - 1)] : 0.0;
#pragma unroll
                        for (int k = 0; k < CN; ++k) {
                            s[k] -= a[h][k] * l;
                            if (anrm < 0.0) ca[k] += in ? fabs(a[h][k]) : 0.0;
                        }
                    }
                }
#pragma unroll
                for (int k = 0; k < CN; ++k) {
                    const double r = Lx.wv[min(c + k * W, n - 1)] + wave_sum(s[k]);
                    if (anrm < 0.0) cmax = fmax(cmax, wave_sum(ca[k]));
                    if (c + k * W < n) {
                        if (lane == 0) Lx.y[c + k * W] = (float)r;
                        rmax = fmax(rmax, fabs(r));
                    }
                }
            }
            block_max3<TB>(rmax, lmax, cmax, red);
            if (anrm < 0.0) anrm = cmax;   // ||A^T||_inf = largest column sum
            if (rmax <= floor_c * anrm * lmax) return true;
            solve_t<float, TB, double>(LU, ld, n, perm, Lx.y, tmp, S);
            double dmax = 0.0, ln = 0.0, unused = 0.0;
            for (int i = tid; i < n; i += TB) {
                const double d = tmp[i];
                lam[i] += d;
                dmax = fmax(dmax, fabs(d));
                ln = fmax(ln, fabs(lam[i]));
            }
            block_max3<TB>(dmax, ln, unused, red);
            if (dmax <= 1e-12 * ln) return true;
        }
        return false;
    }
}

}  // namespace adj
}  // namespace
}  // namespace panel
