// lu_block_impl.hpp -- one workgroup factors one system: batched LU with
// partial pivoting and the back substitution, for systems of up to
// RMAX * TB rows.  Device functions only; the kernels are in lu_block.hip and
// lu_batch.hip.
//
// Sec. 3 of the paper: every airfoil needs the LU decomposition of its dense
// system.  One wavefront per system (lu_wave_impl.hpp) keeps the GPU full
// when there are thousands of small systems; a large system, or a small
// batch, needs the whole workgroup on one system.
//
// Algorithm (right-looking by super-panels of 64 columns, or of two halves of
// 64 whose update of the rest is one of rank 128; LAPACK getrf semantics):
//   * a pivot panel of NB = 16 columns sits in registers, one row per thread
//     (row k0 + tid + TB q in slot q).  Before it is factored it takes the
//     rank-16p update from the super-panel's p panels to its left on the
//     matrix cores: each wavefront updates the rows it owns, and a private
//     LDS tile turns the matrix-core layout into a row per lane, so the
//     updated panel makes no round trip through memory;
//   * pivoting is implicit while the panel is factored (rows stay in their
//     registers, each slot tracks the position its row occupies).  A column
//     costs one barrier: every wavefront publishes its candidate (a 32-bit
//     order-preserving prefix of |a|, resolved exactly on ties) with the
//     candidate's row, and after the barrier each wavefront picks the winner
//     by a reduction over the wavefronts' prefixes;
//   * the row moves of a panel are applied to all other columns as one
//     gather / scatter per column;
//   * the trailing update runs in rounds of 16 NT columns per wavefront: the
//     band rows of those columns are solved in registers (diagonal blocks by
//     their inverses) and stay there as the stationary operand, the
//     super-panel's rows of L stream through a double-buffered LDS tile that
//     all wavefronts share, and the C tiles stream through registers one
//     tile ahead.  L is read once per round instead of once per 16 NT
//     columns.
// The K right-hand sides ride along; the back substitution solves all of
// them in one pass over U.
//
// What bounds it: 256 systems of order 1025 (one per CU) spend two thirds of
// their time in the trailing update, at about half the FP64 matrix rate.  A
// small system waits: one of order 161 (FP64, nine right-hand sides) takes 3140
// cycles per column, 1410 of them in the pivot chain (search, exchange of the
// candidates, rank-1 update), 440 loading panels with their left-looking update,
// 430 storing them, moving rows and gathering the band, 440 in the trailing
// update, 420 in the back substitution.
// Measured (HIP events) against a version with a thread per column for the
// triangular solves, U staged in LDS and one right-hand side per back
// substitution: 14.7 -> 7.03 ms (256 x 1025, FP64, eight right-hand sides), 8.45
// -> 4.57 ms in FP32, 7.60 -> 3.97 ms (1980 systems of 321 to 513, FP32).
#pragma once

#include <climits>

#include "lu_wave_impl.hpp"
#include "panel_internal.hpp"
#include "wave.hpp"

namespace panel {
namespace {
namespace blk {

using wv::TileMap;
using wv::mfma_t;
using wv::opaque_s;

constexpr int NB = 16;          // pivot panel width
constexpr int BSP = 64;         // super-panel width
constexpr int NBK = BSP / NB;   // 16-row blocks of its band
constexpr int RGM = 2;          // most row tiles in flight per LDS buffer

// 32-bit order-preserving prefix of a = |value|: 1 for zero, larger for
// larger values (0: no candidate).  Exact for FP32; for FP64 values that
// share a high word (or lie below its range) share the prefix.
__device__ __forceinline__ unsigned prefix_of(float a) { return (unsigned)__float_as_int(a) + 1u; }
__device__ __forceinline__ unsigned prefix_of(double a) {
    const unsigned hi = (unsigned)__double2hiint(a);
    return (a > 0.0 ? max(hi, 1u) : 0u) + 1u;
}

template <int CTRL> __device__ __forceinline__ unsigned dpp_umax(unsigned v) {
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
    return v > o ? v : o;
}
// Maximum over the 64 lanes, as a scalar.
__device__ __forceinline__ unsigned wave_umax(unsigned v) {
    v = dpp_umax<0xB1>(v);    // quad_perm [1,0,3,2]
    v = dpp_umax<0x4E>(v);    // quad_perm [2,3,0,1]
    v = dpp_umax<0x141>(v);   // row_half_mirror
    v = dpp_umax<0x140>(v);   // row_mirror
    const unsigned a = (unsigned)__builtin_amdgcn_readlane((int)v, 0), b = (unsigned)__builtin_amdgcn_readlane((int)v, 16);
    const unsigned c = (unsigned)__builtin_amdgcn_readlane((int)v, 32), d = (unsigned)__builtin_amdgcn_readlane((int)v, 48);
    return max(max(a, b), max(c, d));
}

// The multipliers a / x of one column step, x the pivot (uniform over the
// workgroup, |a| <= |x|) and kmax its prefix.  FP64: with r the hardware
// estimate (2^-23) after one Newton step, a r corrected by its own remainder,
// which leaves the rounding of the last step (0.5 ulp; a r alone is off by up to
// 1.5); a division costs several times the latency, once per pivot column.
// Where r or a remainder could leave the normal range, the division itself.
template <int R> __device__ __forceinline__ void multipliers(double (&l)[R], double x, unsigned kmax) {
    if (__builtin_expect(kmax > 0x04000000u && kmax <= 0x7bf00000u, 1)) {   // 2^-959 <= |x| < 2^960
        double r = __builtin_amdgcn_rcp(x);
        r = fma(fma(-x, r, 1.0), r, r);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const double t = l[q] * r;
            l[q] = fma(fma(-x, t, l[q]), r, t);
        }
    } else {
#pragma unroll
        for (int q = 0; q < R; ++q) l[q] = l[q] / x;
    }
}
template <int R> __device__ __forceinline__ void multipliers(float (&l)[R], float x, unsigned) {
#pragma unroll
    for (int q = 0; q < R; ++q) l[q] = l[q] / x;
}

// Position of element (row r, column k) of a 16x16 block in the A-operand
// fragment order of the band solve: [lane][k-step].
template <typename T> __device__ __forceinline__ int frag_at(int r, int k) {
    return 4 * ((k & 3) * 16 + TileMap<T>::arow(r)) + (k >> 2);
}
__device__ __forceinline__ constexpr int pair_at(int i2, int i) { return i2 * (i2 + 1) / 2 + i; }

// H: 64-column halves of a super-panel (1 or 2).
template <typename T, int TB, int H = 1> struct BlkLds {
    static constexpr int W = TB / 64, NBT = NBK * H;
    // the super-panel's band in fragment order: inverses of the unit-lower
    // diagonal blocks and the blocks of L below them
    alignas(16) T band[NBT * (NBT + 1) / 2][4 * 64];
    alignas(16) T crow[2][W][NB];     // each wavefront's candidate row (double-buffered)
    unsigned ckey[2][W];              // and its prefix (0: none),
    T cval[2][W];                     // magnitude
    int cpos[2][W];                   // and current position
    alignas(16) T l11[NB][NB];        // unit-lower diagonal block of the panel, by columns
    int mv_src[2 * NB], mv_dst[2 * NB], nmv;   // row moves of the panel
    int ipiv[NB];
    union U {
        T st[W][NB][64];                                  // panel rows in transit (per wavefront)
        alignas(16) T tile[2][RGM][16 * BSP * H];             // L tiles of the trailing update
        struct { T sblk[64 * 64]; T xs[64][NB + 1]; } bs;  // back substitution
    } u;
};

// ---- one column step of the panel factorisation (C is compile-time) --------
template <typename T, int R, int C, int TB, typename Lds>
__device__ __forceinline__ void blk_col(T (&p)[R][NB], int (&pos)[R], unsigned &live, int k0, int &info,
                                        Lds &S) {
    constexpr int buf = C & 1, W = TB / 64;
    constexpr int VW = 16 / (int)sizeof(T), V0 = C / VW;   // 16-byte pieces of a row from the one that holds C
    typedef T vec_t __attribute__((ext_vector_type(VW)));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = k0 + C;
    // this thread's candidate among its rows not yet used as pivots: largest
    // |a|, lowest current position on ties
    T best = T(-1);
    int bq = 0, bpos = INT_MAX;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const T a = fabs(p[q][C]);
        if (((live >> q) & 1u) && (a > best || (R > 1 && a == best && pos[q] < bpos))) {
            best = a;
            bq = q;
            bpos = pos[q];
        }
    }
    const unsigned key = best >= T(0) ? prefix_of(best) : 0u;
    const unsigned wk = wave_umax(key);
    if (wk == 0u) {
        if (lane == 0) S.ckey[buf][wave] = 0u;
    } else {
        unsigned long long m = __ballot(key == wk);
        if (__popcll(m) > 1) {   // rare: equal prefixes, resolved exactly
            const double bd = key == wk ? (double)best : -1.0;
            const double wb = wave_max(bd);
            int cand = bd == wb ? bpos : INT_MAX;
#pragma unroll 1
            for (int off = 32; off > 0; off >>= 1) cand = min(cand, __shfl_xor(cand, off));
            m = __ballot(bd == wb && bpos == cand);
        }
        const int plane = __ffsll((long long)m) - 1;
        const int pq = R > 1 ? __builtin_amdgcn_readlane(bq, plane) : 0;
        if (lane == plane) {
            S.ckey[buf][wave] = wk;
            S.cval[buf][wave] = best;
            S.cpos[buf][wave] = bpos;
#pragma unroll
            for (int q = 0; q < R; ++q)
                if (q == pq) {
#pragma unroll
                    for (int c = V0; c < NB / VW; ++c) {
                        vec_t x;
#pragma unroll
                        for (int e = 0; e < VW; ++e) x[e] = p[q][VW * c + e];
                        *reinterpret_cast<vec_t *>(&S.crow[buf][wave][VW * c]) = x;
                    }
                }
        }
    }
    lds_barrier();
    // the workgroup's pivot: every lane holds one wavefront's prefix
    const unsigned kw = S.ckey[buf][lane & (W - 1)];
    unsigned km = dpp_umax<0x4E>(dpp_umax<0xB1>(kw));
    if constexpr (W > 4) km = dpp_umax<0x141>(km);
    const unsigned kmax = (unsigned)__builtin_amdgcn_readfirstlane((int)km);
    const unsigned wm = (unsigned)__ballot(kw == kmax) & ((1u << W) - 1u);
    int pw = __ffs((int)wm) - 1;
    if (kmax <= 1u) {
        // exact zero pivot (or no finite candidate): LAPACK records the
        // column and leaves it; the row now at position g stays there
        if (info == 0) info = g + 1;
#pragma unroll
        for (int q = 0; q < R; ++q)
            if (pos[q] == g) live &= ~(1u << q);
        if (tid == 0) S.ipiv[C] = g;
        return;
    }
    if ((wm & (wm - 1u)) != 0u) {   // equal prefixes: magnitude, then position
        T bv = T(-1);
        int bp = INT_MAX;
#pragma unroll 1
        for (int w = 0; w < W; ++w)
            if ((wm >> w) & 1u) {
                const T a = S.cval[buf][w];
                const int ps = S.cpos[buf][w];
                if (a > bv || (a == bv && ps < bp)) {
                    bv = a;
                    bp = ps;
                    pw = w;
                }
            }
        pw = __builtin_amdgcn_readfirstlane(pw);
    }
    T u[NB];
#pragma unroll
    for (int c = V0; c < NB / VW; ++c) {
        const vec_t x = *reinterpret_cast<const vec_t *>(&S.crow[buf][pw][VW * c]);
#pragma unroll
        for (int e = 0; e < VW; ++e) u[VW * c + e] = x[e];
    }
    const int ppos = S.cpos[buf][pw];
    T l[R];
#pragma unroll
    for (int q = 0; q < R; ++q) l[q] = p[q][C];
    multipliers<R>(l, u[C], kmax);
    // the pivot row moves to position g (and leaves the candidates), the row
    // at g to the pivot row's position
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int t = pos[q];
        pos[q] = t == ppos ? g : t == g ? ppos : t;
        live = t == ppos ? live & ~(1u << q) : live;
    }
    if (tid == 0) S.ipiv[C] = ppos;
    // rank-1 update of the rows still live; a zero multiplier, not a branch,
    // leaves the others alone (under a branch the compiler copied the whole
    // register array around it)
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const bool lv = (live >> q) & 1u;
        const T lm = lv ? l[q] : T(0);
        p[q][C] = lv ? l[q] : p[q][C];
#pragma unroll
        for (int cc = C + 1; cc < NB; ++cc) p[q][cc] -= lm * u[cc];
    }
}

template <typename T, int R, int C, int TB, typename Lds>
__device__ __forceinline__ void blk_cols(T (&p)[R][NB], int (&pos)[R], unsigned &live, int k0, int nb, int &info,
                                         Lds &S) {
    if constexpr (C < NB) {
        if (C < nb) {
            blk_col<T, R, C, TB>(p, pos, live, k0, info, S);
            blk_cols<T, R, C + 1, TB>(p, pos, live, k0, nb, info, S);
        }
    }
}

// Solve one column block's band in registers: f[4 i + e] holds the band's
// block i in B-operand order (lane l: row 4 e + l/16 of block i, column
// l%16), blocks i < nblk (the band's from i0 on): X_i = linv_i Y_i, then Y_j -= L_ji X_i.
template <typename T, int NT, int NBLK>
__device__ __forceinline__ void band_solve(T (&uf)[NT][4 * NBLK], int nblk, int i0, const T (*band)[4 * 64]) {
    typedef typename TileMap<T>::acc acc_t;
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NBLK; ++i) {
        if (i < nblk) {
            T li[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) li[s] = band[pair_at(i0 + i, i0 + i)][4 * lane + s];
            T xn[NT][4];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc_t acc;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = T(0);
#pragma unroll
                for (int s = 0; s < 4; ++s) acc = mfma_t(li[s], uf[t][4 * i + s], acc);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uf[t][4 * i + e] = acc[e];
                    xn[t][e] = -acc[e];
                    asm volatile("" : "+v"(xn[t][e]));
                }
            }
#pragma unroll
            for (int j = i + 1; j < NBLK; ++j) {
                if (j < nblk) {
                    T lb[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) lb[s] = band[pair_at(i0 + j, i0 + i)][4 * lane + s];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        acc_t acc;
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[e] = uf[t][4 * j + e];
#pragma unroll
                        for (int s = 0; s < 4; ++s) acc = mfma_t(lb[s], xn[t][s], acc);
#pragma unroll
                        for (int e = 0; e < 4; ++e) uf[t][4 * j + e] = acc[e];
                    }
                }
            }
        }
    }
}

// Rows k0.. of the panel's columns into registers (a row per thread and
// slot), after the update from the np panels of the super-panel to the left:
// A[k0:n, panel] -= L[k0:n, K0:k0] U, U = L_band^{-1} A[K0:k0, panel].  Every
// wavefront forms U for itself (no exchange to wait for); the first one
// writes it back, once all have read the band.
template <typename T, int R, int TB, typename Lds>
__device__ __forceinline__ void blk_load(T (&p)[R][NB], T *A, int ld, int n, int K0, int k0, int nb, int np, int i0,
                                         Lds &S) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (np == 0) {
        // every load is issued (clamped addresses) before any is masked
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int rr = min(k0 + tid + TB * q, n - 1);
#pragma unroll
            for (int cc = 0; cc < NB; ++cc) p[q][cc] = A[(size_t)(k0 + min(cc, nb - 1)) * ld + rr];
        }
        __builtin_amdgcn_sched_barrier(0);
        return;
    }
    typedef typename TileMap<T>::acc acc_t;
    constexpr int PM = NBK - 1;         // most panels to the left
    constexpr int HT = R == 1 ? 4 : 2;  // row tiles in flight
    const int i16 = lane & 15, k4 = lane >> 4;
    T uf[1][4 * PM];
    T *up = A + (size_t)(k0 + min(i16, nb - 1)) * ld + K0 + k4;
#pragma unroll
    for (int i = 0; i < PM; ++i)
        if (i < np) {
#pragma unroll
            for (int e = 0; e < 4; ++e) uf[0][4 * i + e] = up[16 * i + 4 * e];
        }
    band_solve<T, 1, PM>(uf, np, i0, S.band);
    lds_barrier();   // every wavefront has read the band (its solve used the loads)
    if (wave == 0 && i16 < nb) {
#pragma unroll
        for (int i = 0; i < PM; ++i)
            if (i < np) {
#pragma unroll
                for (int e = 0; e < 4; ++e) up[16 * i + 4 * e] = uf[0][4 * i + e];
            }
    }
#pragma unroll
    for (int s = 0; s < 4 * PM; ++s) {
        uf[0][s] = -uf[0][s];
        asm volatile("" : "+v"(uf[0][s]));
    }
    T (*st)[64] = S.u.st[wave];
    const T *lcol = A + (size_t)(K0 + k4) * ld;
    const T *ccol[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) ccol[e] = A + (size_t)(k0 + min(TileMap<T>::col(lane, e), nb - 1)) * ld;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int rw = k0 + 64 * wave + TB * q;   // the wavefront's first row of the slot
        if (rw < n) {
#pragma unroll 1
            for (int h = 0; h < 4; h += HT) {
                T lf[HT][4 * PM];
                acc_t acc[HT];
#pragma unroll
                for (int t = 0; t < HT; ++t) {
                    const int r = min(rw + 16 * (h + t) + i16, n - 1);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[t][e] = ccol[e][r];
                }
#pragma unroll
                for (int i = 0; i < PM; ++i)
                    if (i < np) {
#pragma unroll
                        for (int t = 0; t < HT; ++t) {
                            const int r = min(rw + 16 * (h + t) + i16, n - 1);
#pragma unroll
                            for (int e = 0; e < 4; ++e) lf[t][4 * i + e] = lcol[(size_t)(16 * i + 4 * e) * ld + r];
                        }
                    }
#pragma unroll
                for (int i = 0; i < PM; ++i)
                    if (i < np) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int t = 0; t < HT; ++t) acc[t] = mfma_t(uf[0][4 * i + e], lf[t][4 * i + e], acc[t]);
                    }
#pragma unroll
                for (int t = 0; t < HT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) st[TileMap<T>::col(lane, e)][16 * (h + t) + i16] = acc[t][e];
            }
            wv::wave_sync();
        }
#pragma unroll
        for (int cc = 0; cc < NB; ++cc) p[q][cc] = st[cc][lane];   // (rows past n: masked by the caller)
        wv::wave_sync();
    }
}

// ---- one pivot panel: load and update, factorise, store ---------------------
template <typename T, int R, int TB, typename Lds>
__device__ __forceinline__ void blk_panel(T *A, int ld, int n, int K0, int k0, int nb, int i0, int32_t *piv, int &info,
                                          Lds &S) {
    ld = opaque_s(ld);
    const int tid = threadIdx.x;
    T p[R][NB];
    const int np = (k0 - K0) / NB;
    blk_load<T, R, TB>(p, A, ld, n, K0, k0, nb, np, i0, S);
    int pos[R];
    unsigned live = 0;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int r = k0 + tid + TB * q;
        pos[q] = r;
        if (r < n) live |= 1u << q;
#pragma unroll
        for (int cc = 0; cc < NB; ++cc) p[q][cc] = (r < n && cc < nb) ? p[q][cc] : T(0);
    }
    if (tid < NB * NB) (&S.l11[0][0])[tid] = T(0);
    if (tid == 0) S.nmv = 0;

    blk_cols<T, R, 0, TB>(p, pos, live, k0, nb, info, S);

    // rows back at their final positions; the diagonal block to LDS
#pragma unroll
    for (int q = 0; q < R; ++q) {
        const int r = k0 + tid + TB * q;
        if (r < n) {
            T *dst = A + (size_t)k0 * ld + pos[q];
            if (nb == NB) {
#pragma unroll
                for (int cc = 0; cc < NB; ++cc) dst[(size_t)cc * ld] = p[q][cc];
            } else {
#pragma unroll
                for (int cc = 0; cc < NB; ++cc)
                    if (cc < nb) dst[(size_t)cc * ld] = p[q][cc];
            }
            const int d = pos[q] - k0;
            if (d < NB) {
#pragma unroll
                for (int cc = 0; cc < NB; ++cc)
                    if (cc < d) S.l11[cc][d] = p[q][cc];
            }
            if (pos[q] != r) {
                const int idx = atomicAdd(&S.nmv, 1);   // at most two rows move per column
                S.mv_src[idx] = r;
                S.mv_dst[idx] = pos[q];
            }
        }
    }
    __syncthreads();
    if (tid < nb) piv[k0 + tid] = S.ipiv[tid];
}

// The panel's row moves on every column outside it, a column per thread: all
// of a column's loads are issued together, moves past nmv repeat the last.
template <typename T, int M, int TB, typename Lds>
__device__ __forceinline__ void blk_moves_m(T *A, int ld, int ncols, int k0, int nb, int nmv, Lds &S) {
    int src[M], dst[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int mm = min(m, nmv - 1);
        src[m] = S.mv_src[mm];
        dst[m] = S.mv_dst[mm];
    }
#pragma unroll 1
    for (int j = threadIdx.x; j < ncols; j += TB) {
        if (j >= k0 && j < k0 + nb) continue;
        T *cp = A + (size_t)j * ld;
        T t[M];
#pragma unroll
        for (int m = 0; m < M; ++m) t[m] = cp[src[m]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < M; ++m) cp[dst[m]] = t[m];
    }
}

template <typename T, int TB, typename Lds>
__device__ __forceinline__ void blk_moves(T *A, int ld, int ncols, int k0, int nb, Lds &S) {
    const int nmv = __builtin_amdgcn_readfirstlane(S.nmv);
    if (nmv == 0) return;
    ld = opaque_s(ld);
    if (nmv <= 2)
        blk_moves_m<T, 2, TB>(A, ld, ncols, k0, nb, nmv, S);
    else if (nmv <= 8)
        blk_moves_m<T, 8, TB>(A, ld, ncols, k0, nb, nmv, S);
    else
        blk_moves_m<T, 2 * NB, TB>(A, ld, ncols, k0, nb, nmv, S);
}

// Inverse of the panel's unit-lower diagonal block, into the band (one
// wavefront; lane j < 16 solves L x = e_j; each column of L is read from LDS
// while the one before it is used).
template <typename T, int TB, typename Lds>
__device__ __forceinline__ void blk_linv(int i, Lds &S) {
    constexpr int VW = 16 / (int)sizeof(T);
    typedef T vec_t __attribute__((ext_vector_type(VW)));
    const int lane = threadIdx.x & 63;
    if (lane < NB) {
        T x[NB];
        vec_t l[2][NB / VW];
#pragma unroll
        for (int r = 0; r < NB; ++r) x[r] = (r == lane) ? T(1) : T(0);
#pragma unroll
        for (int c = 0; c < NB / VW; ++c) l[0][c] = reinterpret_cast<const vec_t *>(&S.l11[0][0])[c];
#pragma unroll
        for (int cc = 0; cc < NB - 1; ++cc) {
            if (cc + 1 < NB - 1) {
#pragma unroll
                for (int c = (cc + 2) / VW; c < NB / VW; ++c)
                    l[(cc + 1) & 1][c] = reinterpret_cast<const vec_t *>(&S.l11[cc + 1][0])[c];
            }
            const T xc = x[cc];
#pragma unroll
            for (int r = cc + 1; r < NB; ++r) x[r] -= l[cc & 1][r / VW][r % VW] * xc;
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int r = 0; r < NB; ++r) S.band[pair_at(i, i)][frag_at<T>(r, lane)] = x[r];
    }
}

// TileMap::col as lane * (lane group) + step * element.
template <typename T> struct ColMap;
template <> struct ColMap<double> { static constexpr int lane = 1, step = 4; };
template <> struct ColMap<float> { static constexpr int lane = 4, step = 1; };

// ---- trailing update ---------------------------------------------------------
// One round: 16 NT columns per column group of wavefronts, starting at cs0
// (columns up to c1); RG row groups of wavefronts share each column group.
//   U  = L_band^{-1} A[band, columns]          (band: nblk 16-row blocks at kb)
//   A[kend:n, columns] -= A[kend:n, band] U    (kend < n: the band is full)
template <typename T, int TB, int NT, int RG, int NBLK, typename Lds>
__device__ __forceinline__ void blk_round(T *A, int ld, int n, int kb, int kend, int cs0, int c1, int nblk,
                                          Lds &S) {
    constexpr int W = TB / 64, WC = W / RG, S4 = 4 * NBLK;
    constexpr int VW = 16 / (int)sizeof(T);      // k-steps per 16-byte LDS read
    constexpr int E = RG * 16 * 16 * NBLK / TB;        // staged elements per thread
    typedef typename TileMap<T>::acc acc_t;
    typedef T vec_t __attribute__((ext_vector_type(VW)));
    ld = opaque_s(ld);
    const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, k4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = wave % WC, rg = wave / WC;
    const int cs = cs0 + 16 * NT * cg;
    const bool act = cs < c1;   // wave-uniform: this wavefront has columns
    T uf[NT][S4];
    if (act) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const T *up = A + (size_t)min(cs + 16 * t + i16, c1 - 1) * ld + kb + k4;
#pragma unroll
            for (int s = 0; s < S4; ++s) uf[t][s] = (s < 4 * nblk) ? up[4 * s] : T(0);
        }
        band_solve<T, NT, NBLK>(uf, nblk, 0, S.band);
    }
    if constexpr (RG > 1) lds_barrier();   // the other row groups have read the band
    if (act && rg == 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int c = cs + 16 * t + i16;
            if (c < c1) {
                T *up = A + (size_t)c * ld + kb + k4;
#pragma unroll
                for (int s = 0; s < S4; ++s)
                    if (s < 4 * nblk) up[4 * s] = uf[t][s];
            }
        }
    }
    if (kend >= n) return;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int s = 0; s < S4; ++s) {
            uf[t][s] = -uf[t][s];
            asm volatile("" : "+v"(uf[t][s]));
        }
    // C columns of this lane, col(lane, e) = lane part + uniform part.  In FP32
    // and in the rank-128 rounds, a round of whole columns reads each (t, e) at
    // a scalar base plus one per-lane offset, which saves two or three vector
    // instructions per access (256 x 1025 in FP64: 7.50 -> 7.03 ms; 1980 systems
    // of 321 to 513 in FP32: 4.10 -> 3.97); the other FP64 rounds keep an element
    // offset per column (256 x 513: 1.49 ms against 1.57 at scalar bases).
    constexpr bool SB = sizeof(T) == 4 || NBLK > NBK;
    constexpr int LC = ColMap<T>::lane, UC = ColMap<T>::step;
    const bool whole = SB && cs + 16 * NT <= c1;   // wave-uniform
    const char *cbase = reinterpret_cast<const char *>(A + (size_t)min(cs, c1 - 1) * ld);
    const unsigned clane = (unsigned)(LC * k4 * ld) * (unsigned)sizeof(T);
    auto cptr = [&](int t, int e, int r) {
        return reinterpret_cast<T *>(const_cast<char *>(cbase) + (size_t)((16 * t + UC * e) * ld) * sizeof(T) +
                                     (clane + (unsigned)r * (unsigned)sizeof(T)));
    };
    int coff[SB ? 1 : NT][4];
    bool cok[SB ? 1 : NT][4];
    if constexpr (!SB) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = cs + 16 * t + LC * k4 + UC * e;
                cok[t][e] = c < c1;
                coff[t][e] = min(c, c1 - 1) * ld;
            }
    }
    auto ccol = [&](int t, int e) { return cs + 16 * t + LC * k4 + UC * e; };
    // element (r, c) for a load of a round that runs past c1: in FP32 with
    // rank-64 updates by a 32-bit offset from the system's base (a system is less
    // than 2^23 bytes), whose registers the C tile of the next step leaves free
    // (uneven batch of 4096, FP32 step: 7.78 -> 7.57 ms with the stores addressed
    // by pointers all the same)
    auto cedge = [&](int c, int r) {
        if constexpr (NBLK == NBK)
            return reinterpret_cast<T *>(reinterpret_cast<char *>(A) + (unsigned)(c * ld + r) * (unsigned)sizeof(T));
        else
            return A + ((size_t)c * ld + r);
    };
    // staging: thread tid brings elements tid + TB e of a 16 RG x 16 NBLK tile
    // (rows fastest) into fragment order
    const int nit = (n - kend + 16 * RG - 1) / (16 * RG);
    const int sr = tid % (16 * RG), sk = tid / (16 * RG);
    constexpr int KS = TB / (16 * RG);   // columns between a thread's elements
    const T *lsrc = A + (size_t)(kb + sk) * ld;
    T lreg[E];
    auto load_l = [&](int it) {
        const int r = min(kend + 16 * RG * it + sr, n - 1);
#pragma unroll
        for (int e = 0; e < E; ++e) lreg[e] = lsrc[(size_t)(KS * e) * ld + r];
    };
    auto store_l = [&](int buf) {
        T *dst = &S.u.tile[buf][sr >> 4][0];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = sk + KS * e, s = k >> 2;
            dst[((s / VW) * 64 + (k & 3) * 16 + (sr & 15)) * VW + s % VW] = lreg[e];
        }
    };
    T cb[NT][4];
    auto load_c = [&](int it) {
        const int r = min(kend + 16 * (RG * it + rg) + i16, n - 1);
        if (whole) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) cb[t][e] = *cptr(t, e, r);
        } else {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (SB)
                        cb[t][e] = *cedge(min(ccol(t, e), c1 - 1), r);
                    else
                        cb[t][e] = A[coff[t][e] + r];
                }
            }
        }
    };
    load_l(0);
    store_l(0);
    load_l(1);
    if (act) load_c(0);
#pragma unroll 1
    for (int it = 0; it < nit; ++it) {
        lds_barrier();   // buffer it & 1 is filled, the other one is free
        if (it + 1 < nit) store_l((it + 1) & 1);
        load_l(it + 2);
        if (act) {
            // C starts the sums: the first products take it down to the size of
            // the Schur complement, which is far smaller for these smooth
            // kernels, and the rounding of the others follows it down.  (Sums
            // from zero with C added after them round at C's size throughout: the
            // solutions of order 1025 were off by 2.5e-11 instead of 7e-13, of
            // order 401 by 2.1e-12 instead of 1.6e-13, FP32 before refinement
            // 6.3e-3 and 1.2e-3 instead of 8.6e-4 and 1.6e-4.)
            acc_t acc[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][e] = cb[t][e];
            load_c(it + 1);   // (ahead of the products: 256 x 1025, FP64: 7.52 -> 7.07 ms)
            const vec_t *lt = reinterpret_cast<const vec_t *>(&S.u.tile[it & 1][rg][0]) + lane;
#pragma unroll
            for (int sv = 0; sv < S4 / VW; ++sv) {
                const vec_t lf = lt[sv * 64];
#pragma unroll
                for (int w = 0; w < VW; ++w)
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t] = mfma_t(uf[t][sv * VW + w], lf[w], acc[t]);
            }
            const int r = kend + 16 * (RG * it + rg) + i16;
            if (r < n) {
                if (whole) {
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e) *cptr(t, e, r) = acc[t][e];
                } else {
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if constexpr (SB) {
                                if (ccol(t, e) < c1) A[(size_t)ccol(t, e) * ld + r] = acc[t][e];
                            } else {
                                if (cok[t][e]) A[coff[t][e] + r] = acc[t][e];
                            }
                }
            }
        }
    }
    lds_barrier();   // the tiles are free again
}

template <typename T, int TB, int RG, int NT, int NBLK, typename Lds>
__device__ __forceinline__ void blk_rounds(int nt, T *A, int ld, int n, int kb, int kend, int c0, int c1, int nblk,
                                           Lds &S) {
    if constexpr (NT >= 1) {
        if (nt == NT) {
#pragma unroll 1
            for (int cs = c0; cs < c1; cs += 16 * NT * (TB / 64 / RG))
                blk_round<T, TB, NT, RG, NBLK>(A, ld, n, kb, kend, cs, c1, nblk, S);
        } else {
            blk_rounds<T, TB, RG, NT - 1, NBLK>(nt, A, ld, n, kb, kend, c0, c1, nblk, S);
        }
    }
}

// Columns [c0, c1) right of the super-panel kb..kend.
// NTM: largest number of 16-column tiles per wavefront and round, as many as
// the instance's registers hold next to the C tiles in flight.
template <typename T, int TB, int NTM, int NBLK, typename Lds>
__device__ __forceinline__ void blk_update(T *A, int ld, int n, int kb, int kend, int c0, int c1, Lds &S) {
    constexpr int W = TB / 64;
    const int nblk = (kend - kb + NB - 1) / NB;
    const int ct = (c1 - c0 + 15) / 16, rt = (n - kend + 15) / 16;
    // fewest products on the longest wavefront, one row group or two: rounds
    // x tiles per wavefront x row tiles, with the band solve counted as the
    // 16-row products it is
    constexpr int BS = NBLK * (NBLK + 1) / 2;
    const int r1 = (ct + W * NTM - 1) / (W * NTM), n1 = (ct + r1 * W - 1) / (r1 * W);
    const int r2 = (ct + W / 2 * NTM - 1) / (W / 2 * NTM), n2 = (ct + r2 * (W / 2) - 1) / (r2 * (W / 2));
    if (r1 * n1 * (NBLK * rt + BS) <= r2 * n2 * (NBLK / 2 * (rt + 1) + BS))
        blk_rounds<T, TB, 1, NTM, NBLK>(n1, A, ld, n, kb, kend, c0, c1, nblk, S);
    else
        blk_rounds<T, TB, 2, NTM, NBLK>(n2, A, ld, n, kb, kend, c0, c1, nblk, S);
}

// The diagonal block of the back substitution: lane = row, up to NR
// right-hand sides side by side in a wavefront.
template <typename T, int TB, int NR, typename Lds>
__device__ __forceinline__ void blk_diag(int n, int K, int rb, int w, double *X, Lds &S) {
    constexpr int W = TB / 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wave >= K) return;
    const T *sblk = S.u.bs.sblk;
    T yi[NR];
#pragma unroll
    for (int m = 0; m < NR; ++m)
        yi[m] = lane < w ? (T)X[(size_t)min(wave + W * m, K - 1) * n + rb + lane] : T(0);
    const T dinv = lane < w ? T(1) / sblk[lane * 64 + lane] : T(0);
#pragma unroll 1
    for (int j0 = 56; j0 >= 0; j0 -= 8) {
        if (j0 >= w) continue;
        T uj[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) uj[j] = sblk[(j0 + j) * 64 + lane];
#pragma unroll
        for (int j = 7; j >= 0; --j) {
            if (j0 + j < w) {
#pragma unroll
                for (int m = 0; m < NR; ++m) {
                    if (lane == j0 + j) yi[m] *= dinv;
                    const T xj = readlane_t(yi[m], j0 + j);
                    if (lane < j0 + j) yi[m] -= uj[j] * xj;
                }
            }
        }
    }
#pragma unroll
    for (int m = 0; m < NR; ++m) {
        const int k = wave + W * m;
        if (k < K) {
            S.u.bs.xs[lane][k] = yi[m];
            if (lane < w) X[(size_t)k * n + rb + lane] = (double)yi[m];
        }
    }
}

// ---- back substitution U X = Y for all right-hand sides ----------------------
// Y: the columns n..n+K-1 of the system, copied to X (the columns themselves
// keep L^{-1} P b), whose values are held to T's precision.  64-row blocks from the bottom: the
// diagonal block in LDS, one right-hand side per wavefront at a time (lane =
// row), then the rows above take the block's contribution on the matrix
// cores, all right-hand sides at once (U is read once).
template <typename T, int TB, typename Lds>
__device__ __forceinline__ void blk_back(const T *A, int ld, int n, int K, double *X, Lds &S) {
    constexpr int W = TB / 64;
    typedef typename TileMap<T>::acc acc_t;
    ld = opaque_s(ld);
    const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, k4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    T *sblk = S.u.bs.sblk;
    T (*xs)[NB + 1] = S.u.bs.xs;
    for (int idx = tid; idx < 64 * (NB + 1); idx += TB) (&xs[0][0])[idx] = T(0);
#pragma unroll 4
    for (int k = 0; k < K; ++k)
        for (int i = tid; i < n; i += TB) X[(size_t)k * n + i] = (double)A[(size_t)(n + k) * ld + i];
    for (int rb = ((n - 1) / 64) * 64; rb >= 0; rb -= 64) {
        const int w = min(64, n - rb);
        // the block's upper triangle (an entry outside it repeats one inside;
        // the solve below never uses it)
        T d[64 * 64 / TB];
#pragma unroll
        for (int m = 0; m < 64 * 64 / TB; ++m) {
            const int c = min((tid >> 6) + m * W, w - 1), r = min(lane, c);
            d[m] = A[(size_t)(rb + c) * ld + rb + r];
        }
#pragma unroll
        for (int m = 0; m < 64 * 64 / TB; ++m) sblk[tid + m * TB] = d[m];
        __syncthreads();
        const int nr = (K + W - 1) / W;   // right-hand sides per wavefront, solved side by side
        if (nr == 1)
            blk_diag<T, TB, 1>(n, K, rb, w, X, S);
        else if (nr == 2)
            blk_diag<T, TB, 2>(n, K, rb, w, X, S);
        else
            blk_diag<T, TB, 4>(n, K, rb, w, X, S);
        __syncthreads();
        // rows above, a 16-row tile per wavefront at a time
        T xa[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) xa[s] = -xs[4 * s + k4][i16];
        int coff[4];
        bool cok[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = TileMap<T>::col(lane, e);
            cok[e] = c < K;
            coff[e] = min(c, K - 1) * n;
        }
        // columns past a short last block repeat its last one (times zero)
        T lf[16];
        auto load_l = [&](int rt) {
            const int r = min(rt, rb / 16 - 1) * 16 + i16;
#pragma unroll
            for (int s = 0; s < 16; ++s) lf[s] = A[(size_t)(rb + min(4 * s + k4, w - 1)) * ld + r];
        };
        if (rb > 0) load_l(wave);
#pragma unroll 1
        for (int rt = wave; rt < rb / 16; rt += W) {
            const int r = 16 * rt + i16;
            T c0[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) c0[e] = (T)X[coff[e] + r];
            acc_t a0, a1;
#pragma unroll
            for (int e = 0; e < 4; ++e) a0[e] = a1[e] = T(0);
#pragma unroll
            for (int s = 0; s < 16; s += 2) {
                a0 = mfma_t(xa[s], lf[s], a0);
                a1 = mfma_t(xa[s + 1], lf[s + 1], a1);
            }
            load_l(rt + W);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (cok[e]) X[coff[e] + r] = (double)(c0[e] + (a0[e] + a1[e]));
        }
        __syncthreads();
    }
}

// Factor airfoil b's system in place and solve its K right-hand sides, one
// workgroup of TB threads; systems of more than max_n (at most RMAX * TB) rows
// are refused.
template <typename T, int TB, int RMAX, int NTM, int H = 1, typename Lds>
__device__ __forceinline__ void blk_lu(const WsView &v, int b, int max_n, int32_t *__restrict__ info_out, Lds &S) {
    const AirfoilMeta mt = v.meta[b];
    const int n = mt.n1, ld = mt.ld, ncols = mt.n1 + mt.K;
    const int tid = threadIdx.x;
    double *X = v.x + mt.x_off;
    if (v.flag[b] != 0 || n > max_n) {
        // screened out by the assembly (-1), or a system too large for its
        // place in the order (-3: the workspace's airfoil order does not match
        // the plan it is used with)
        const int code = v.flag[b] != 0 ? -1 : -3;
        __syncthreads();
        if (tid == 0) {
            info_out[b] = code;
            v.flag[b] = code;
        }
        for (int i = tid; i < n * mt.K; i += TB) X[i] = __builtin_nan("");
        return;
    }
    T *A = wv::sys_of<T>(v, mt);
    int32_t *piv = v.piv + mt.piv_off;
    int info = 0;
    // super-panels of H halves of 64 columns: with H = 2 the first half updates
    // the second one only, and the columns to the right of both take one
    // rank-128 update
    for (int KS = 0; KS < n; KS += BSP * H) {
        const int ks1 = min(KS + BSP * H, n);
#pragma unroll 1
        for (int K0 = KS; K0 < ks1; K0 += BSP) {
            const int kend = min(K0 + BSP, n), i0 = (K0 - KS) / NB;
            for (int k0 = K0; k0 < kend; k0 += NB) {
                const int nb = min(NB, n - k0), i = (k0 - KS) / NB;
                const int rows = (n - k0 + TB - 1) / TB;
                if (rows == 1)
                    blk_panel<T, 1, TB>(A, ld, n, K0, k0, nb, i0, piv, info, S);
                else if (RMAX == 2 || rows == 2)
                    blk_panel<T, 2, TB>(A, ld, n, K0, k0, nb, i0, piv, info, S);
                else
                    blk_panel<T, (RMAX > 2 ? RMAX : 2), TB>(A, ld, n, K0, k0, nb, i0, piv, info, S);
                blk_moves<T, TB>(A, ld, ncols, k0, nb, S);
                if (tid >= TB - 64) blk_linv<T, TB>(i, S);
                __syncthreads();
                // block row i of the band (its rows are final now)
                for (int idx = tid; idx < 256 * i; idx += TB) {
                    const int r = idx & 15, k = idx >> 4;   // k: column within the band
                    S.band[pair_at(i, k >> 4)][frag_at<T>(r, k & 15)] = A[(size_t)(KS + k) * ld + k0 + r];
                }
                __syncthreads();
            }
            if (H == 2 && i0 == 0 && kend < ks1) {
                blk_update<T, TB, NTM, NBK>(A, ld, n, K0, kend, kend, ks1, S);
                __syncthreads();
            }
        }
        blk_update<T, TB, NTM, NBK * H>(A, ld, n, KS, ks1, ks1, ncols, S);   // (the right-hand sides at least)
        __syncthreads();
    }
    if (tid == 0) {
        info_out[b] = info;
        v.flag[b] = info;
    }
    if (info != 0) {
        for (int i = tid; i < n * mt.K; i += TB) X[i] = __builtin_nan("");
        return;
    }
    blk_back<T, TB>(A, ld, n, mt.K, X, S);
}

}  // namespace blk
}  // namespace
}  // namespace panel
