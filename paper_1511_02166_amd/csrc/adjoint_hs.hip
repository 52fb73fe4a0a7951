// adjoint_hs.hip -- shape gradient in the Hess-Smith formulation.
//
// Unknowns x = (q_0..q_{N-1}, g): source densities and the shared vortex
// density; surface speed u = T x + V_inf e.t (T: the tangential matrix kept
// by the assembly), Cl = -2 sum_j u_j L_j / (V_inf c), Cp_j = 1 - u_j^2/V_inf^2.
// For each angle, with g_j = dF/du_j, w = T^T g and lambda = M^{-T} w, the
// source-block entries A_ji (normal) and T_ji (tangential), i != j, carry the
// weights
//   W_A(j,i) = g_j x_N - lambda_j x_i - k_j lambda_N x_N
//   W_T(j,i) = g_j x_i + lambda_j x_N - k_j lambda_N x_i
// (k_j = 1 on the two trailing-edge rows that form the Kutta row; the
// vortex columns are row sums of the source blocks, so their derivatives
// fold into these weights).  A and T depend on d1 = m_j - P_i, d2 = m_j -
// P_{i+1} through lg = log(|d1|/|d2|) and the subtended angle beta, and on
// the panel angles through c = t_i.t_j = cos(phi_j - phi_i), s = t_i x t_j:
//   d/dd1 (W_A A + W_T T) = (a d1 + b perp(d1)) / (2 pi |d1|^2)
//   d/dd2 (W_A A + W_T T) = -(a d2 + b perp(d2)) / (2 pi |d2|^2)
//   d/dphi_j = -d/dphi_i  = (lg b - beta a) / 2pi
// with a = W_A s + W_T c, b = W_A c - W_T s, perp(v) = (-v_y, v_x).  The
// right-hand sides (-V_inf e.n_j, and -V_inf e.(t_0 + t_{N-1}) on the Kutta
// row), the free-stream part of u and the panel lengths in Cl add explicit
// terms.  Self entries (A_jj = 1/2, T_jj = 0) are constants.
// One workgroup per airfoil takes its angles KA at a time.  The weights W_A and
// W_T of an entry are sums over the angles and everything that follows is
// linear in them, so a group of angles shares one evaluation of each pair's
// logarithms and arctangent.  Pass 1 (a thread per row j and range of panels)
// sums the control-point and row-angle terms; pass 2 (a thread per node k and
// range of rows) sums the endpoint terms of the panels starting and ending at
// node k and the column-angle term of panel k.  The ranges split a row (or
// node) over the threads that a small section would leave idle; their partial
// sums meet in LDS in a fixed order.  Gradients w.r.t. the midpoints (gm) and
// the panel vectors (gh = dF/dphi perp(t)/L + length terms) reach the nodes at
// the end.
//
// What bounds it: FP64 vector arithmetic.  Measured against an evaluation per
// angle and a thread per row or node (HIP events): 96 sections of order 181, two
// angles with Cp cotangents, FP32 factors 0.99 -> 0.36 ms; 1024 of order 257, one
// angle 4.31 -> 2.02 ms (FP32 factors), 2.75 -> 1.52 ms (FP64).
#include "adjoint_impl.hpp"

namespace panel {
namespace {

using namespace adj;

constexpr double kInv2Pi = 0.15915494309189535;
constexpr int KA = 2;   // angles per pair evaluation (their vectors must fit in LDS)

template <typename T, int TB, int NM> struct HsLds {
    double sx[NM], sy[NM];
    double xk[KA][NM], lam[KA][NM], gu[KA][NM];
    double gmx[NM], gmy[NM], ghx[NM], ghy[NM], gnx[NM], gny[NM];
    double tmp[NM];
    union {
        SolveLds<T, TB> solve;
        double part[3][TB];   // partial sums of the ranges
    };
    LambdaLds<T, NM> lx;
    double red[3][TB / 64];
    double at[fm::kAtanTab];
    unsigned short perm[NM];
};

template <typename T, int TB, int NM>
__global__ __launch_bounds__(TB) void adjoint_hs_kernel(WsView v, const double *__restrict__ xy,
                                                        const double *__restrict__ dcl,
                                                        const double *__restrict__ dcp, double *__restrict__ dxy,
                                                        int32_t *__restrict__ info) {
    constexpr int W = TB / 64;
    const int b = v.order[blockIdx.x];
    const AirfoilMeta mt = v.meta[b];
    const int N = mt.N, n1 = mt.n1, K = mt.K, ld = mt.ld;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    double *out = dxy + 2 * (size_t)mt.node_off;
    if (v.flag[b] != 0 || n1 > NM) {
        for (int k = tid; k < 2 * (N + 1); k += TB) out[k] = __builtin_nan("");
        if (info && tid == 0) info[b] = v.flag[b] != 0 ? v.flag[b] : -3;
        return;
    }
    __shared__ HsLds<T, TB, NM> S;
    load_atan_table(S.at);
    const double *P = xy + 2 * (size_t)mt.node_off;
    for (int k = tid; k <= N; k += TB) {
        S.sx[k] = P[2 * k];
        S.sy[k] = P[2 * k + 1];
        S.gnx[k] = S.gny[k] = S.gmx[k] = S.gmy[k] = S.ghx[k] = S.ghy[k] = 0.0;
    }
    perm_of_pivots(v.piv + mt.piv_off, n1, TB, S.perm);
    const double vinf = v.hdr->vinf, chord = v.chord[b];
    const double lscale = -2.0 / (vinf * chord), cpf = -2.0 / (vinf * vinf);
    const PanelGeom *geo = v.geom + mt.panel_off;
    const double *Tg = v.tg + mt.a_off;
    // thread (row or node r, range s) of pass 1, pass 2 and u: s < ns ranges
    // of `len` entries; sections of more than TB rows take several rounds
    const int np = (N + 1 + 63) & ~63;
    const int ns = np < TB ? TB / np : 1;
    const int rs = ns > 1 ? tid / np : 0, r0 = ns > 1 ? tid % np : tid;
    const int len = (N + ns - 1) / ns, e0 = min(rs * len, N), e1 = rs < ns ? min(e0 + len, N) : e0;
    bool conv = true;

    // adds the ranges' partial sums of row r0 into those of range 0 (all
    // threads; nothing to do for a single range)
    auto reduce3 = [&](double &a, double &c, double &d) {
        if (ns == 1) return;
        __syncthreads();
        S.part[0][tid] = a;
        S.part[1][tid] = c;
        S.part[2][tid] = d;
        __syncthreads();
        if (rs == 0) {
            for (int s = 1; s < ns; ++s) {
                a += S.part[0][s * np + r0];
                c += S.part[1][s * np + r0];
                d += S.part[2][s * np + r0];
            }
        }
    };

    for (int k0 = 0; k0 < K; k0 += KA) {
        const int kn = min(KA, K - k0);
        double ex[KA], ey[KA], dk[KA];
#pragma unroll
        for (int k = 0; k < KA; ++k) {
            const int ka = mt.alpha_off + k0 + min(k, kn - 1);
            const double al = v.alpha[ka];
            ex[k] = cos(al);
            ey[k] = sin(al);
            dk[k] = dcl[ka];
            // (an angle past the last counts as zero everywhere)
            for (int i = tid; i < n1; i += TB)
                S.xk[k][i] = k < kn ? v.x[mt.x_off + (size_t)(k0 + k) * n1 + i] : 0.0;
        }
        __syncthreads();
        // u_j = (T x)_j + V_inf e.t_j; g_j = dF/du_j; explicit length term
        for (int j0 = 0; j0 < np; j0 += ns > 1 ? np : TB) {
            const int j = j0 + r0, jc = min(j, N - 1);
            double u[KA] = {}, unused = 0.0;
            const int c1 = rs == ns - 1 ? n1 : e1;   // the last range takes the vortex column too
#pragma unroll 8
            for (int i = e0; i < c1; ++i) {
                const double t = Tg[(size_t)i * ld + jc];
#pragma unroll
                for (int k = 0; k < KA; ++k) u[k] += t * S.xk[k][i];
            }
            static_assert(KA == 2, "reduce3 carries two sums here");
            reduce3(u[0], u[1], unused);
            if (rs == 0 && j < N) {
                const PanelGeom g = geo[j];
                double hx = 0.0, hy = 0.0;
#pragma unroll
                for (int k = 0; k < KA; ++k) {
                    double gj = 0.0;
                    if (k < kn) {
                        const double uj = vinf * (ex[k] * g.tx + ey[k] * g.ty) + u[k];
                        gj = dk[k] * lscale * g.L;
                        if (dcp) gj += dcp[mt.s_off + (size_t)(k0 + k) * N + j] * cpf * uj;
                        const double el = dk[k] * lscale * uj;
                        hx += el * g.tx;
                        hy += el * g.ty;
                    }
                    S.gu[k][j] = gj;
                }
                S.ghx[j] += hx;
                S.ghy[j] += hy;
            }
        }
        __syncthreads();
        for (int k = 0; k < kn; ++k) {
            // w = T^T g: a wavefront per column, lanes along the rows
            for (int c = wave; c < n1; c += 4 * W) {
                double s[4];
                column_dots<double, 4>(Tg, ld, c, W, n1, 0, N, S.gu[k], s);
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    if (lane == 0 && c + m * W < n1) S.tmp[c + m * W] = s[m];
            }
            __syncthreads();
            conv = solve_lambda<T, TB, NM>(v, mt, S.perm, S.lam[k], S.tmp, S.solve, S.lx, S.red) && conv;
            __syncthreads();
        }
        for (int k = kn; k < KA; ++k)
            for (int i = tid; i < n1; i += TB) S.lam[k][i] = 0.0;
        __syncthreads();
        double xN[KA], lN[KA];
#pragma unroll
        for (int k = 0; k < KA; ++k) {
            xN[k] = S.xk[k][N];
            lN[k] = S.lam[k][N];
        }

        // ---- pass 1: rows j -----------------------------------------------
        for (int j0 = 0; j0 < np; j0 += ns > 1 ? np : TB) {
            const int j = j0 + r0, jc = min(j, N - 1);
            const PanelGeom gj = geo[jc];
            const double mx = 0.5 * (S.sx[jc] + S.sx[jc + 1]), my = 0.5 * (S.sy[jc] + S.sy[jc + 1]);
            double WA0 = 0.0, WT0 = 0.0, wa1[KA], wt1[KA];   // the parts of W_A, W_T free of x_i, the factors of x_i
            double erow = 0.0;                               // explicit part of dF/dphi_j
#pragma unroll
            for (int k = 0; k < KA; ++k) {
                const double g = S.gu[k][jc], lj = S.lam[k][jc], kl = (jc == 0 || jc == N - 1) ? lN[k] : 0.0;
                WA0 += g * xN[k] - kl * xN[k];
                WT0 += lj * xN[k];
                wa1[k] = -lj;
                wt1[k] = g - kl;
                const double et = ex[k] * gj.tx + ey[k] * gj.ty, ep = -ex[k] * gj.ty + ey[k] * gj.tx;
                erow += -lj * vinf * et + g * vinf * ep - kl * vinf * ep;
            }
            double ax = 0.0, ay = 0.0, phi = 0.0;
            double d1x = mx - S.sx[e0], d1y = my - S.sy[e0];
            double q1 = d1x * d1x + d1y * d1y, l1 = plog(q1), r1 = pdiv(1.0, q1);
            for (int i = e0; i < e1; ++i) {
                const double d2x = mx - S.sx[i + 1], d2y = my - S.sy[i + 1];
                const double q2 = d2x * d2x + d2y * d2y, l2 = plog(q2), r2 = pdiv(1.0, q2);
                if (i != jc) {
                    const PanelGeom gi = geo[i];
                    const double c = gi.tx * gj.tx + gi.ty * gj.ty, s = gi.tx * gj.ty - gi.ty * gj.tx;
                    double WA = WA0, WT = WT0;
#pragma unroll
                    for (int k = 0; k < KA; ++k) {
                        const double xi = S.xk[k][i];
                        WA += wa1[k] * xi;
                        WT += wt1[k] * xi;
                    }
                    const double aa = WA * s + WT * c, bb = WA * c - WT * s;
                    // (a d + b perp(d)) / |d|^2 at d1, minus the same at d2
                    ax += (aa * d1x - bb * d1y) * r1 - (aa * d2x - bb * d2y) * r2;
                    ay += (aa * d1y + bb * d1x) * r1 - (aa * d2y + bb * d2x) * r2;
                    const double cr = d1x * d2y - d1y * d2x, dd = d1x * d2x + d1y * d2y;
                    const double beta = patan2(-cr, dd, S.at), lg = 0.5 * (l1 - l2);
                    phi += lg * bb - beta * aa;
                }
                d1x = d2x;
                d1y = d2y;
                r1 = r2;
                l1 = l2;
            }
            reduce3(ax, ay, phi);
            if (rs == 0 && j < N) {
                S.gmx[j] += kInv2Pi * ax;
                S.gmy[j] += kInv2Pi * ay;
                // dF/dphi_j: matrix rows, right-hand side, free stream in u
                const double f = (kInv2Pi * phi + erow) / gj.L;
                S.ghx[j] += -f * gj.ty;
                S.ghy[j] += f * gj.tx;
            }
        }
        __syncthreads();   // (pass 2 adds to gh as well)

        // ---- pass 2: nodes --------------------------------------------------
        for (int n0 = 0; n0 < np; n0 += ns > 1 ? np : TB) {
            const int kn0 = n0 + r0, nd = min(kn0, N);
            const double px = S.sx[nd], py = S.sy[nd];
            const bool has_s = nd < N, has_e = nd >= 1;   // panel nd starts / panel nd - 1 ends here
            PanelGeom gs{}, ge{};
            double qx = px, qy = py, xs[KA] = {}, xe[KA] = {};
            if (has_s) {
                gs = geo[nd];
                qx = S.sx[nd + 1];
                qy = S.sy[nd + 1];
            }
            if (has_e) ge = geo[nd - 1];
#pragma unroll
            for (int k = 0; k < KA; ++k) {
                if (has_s) xs[k] = S.xk[k][nd];
                if (has_e) xe[k] = S.xk[k][nd - 1];
            }
            double ex1 = 0.0, ey1 = 0.0, cphi = 0.0;
            for (int j = e0; j < e1; ++j) {
                const PanelGeom gj = geo[j];
                const double mx = 0.5 * (S.sx[j] + S.sx[j + 1]), my = 0.5 * (S.sy[j] + S.sy[j + 1]);
                const bool te = j == 0 || j == N - 1;
                double WA0 = 0.0, WT0 = 0.0, was = 0.0, wts = 0.0, wae = 0.0, wte = 0.0;
#pragma unroll
                for (int k = 0; k < KA; ++k) {
                    const double g = S.gu[k][j], lj = S.lam[k][j], h = g - (te ? lN[k] : 0.0);
                    WA0 += h * xN[k];
                    WT0 += lj * xN[k];
                    was -= lj * xs[k];
                    wts += h * xs[k];
                    wae -= lj * xe[k];
                    wte += h * xe[k];
                }
                const double dx = mx - px, dy = my - py;
                const double q = dx * dx + dy * dy, rq = pdiv(1.0, q);
                if (has_s && j != nd) {   // node nd is P_i of panel i = nd: -d/dd1
                    const double c = gs.tx * gj.tx + gs.ty * gj.ty, s = gs.tx * gj.ty - gs.ty * gj.tx;
                    const double WA = WA0 + was, WT = WT0 + wts;
                    const double aa = WA * s + WT * c, bb = WA * c - WT * s;
                    ex1 -= (aa * dx - bb * dy) * rq;
                    ey1 -= (aa * dy + bb * dx) * rq;
                    const double d2x = mx - qx, d2y = my - qy;
                    const double q2 = d2x * d2x + d2y * d2y;
                    const double cr = dx * d2y - dy * d2x, dd = dx * d2x + dy * d2y;
                    const double beta = patan2(-cr, dd, S.at), lg = 0.5 * (plog(q) - plog(q2));
                    cphi += lg * bb - beta * aa;
                }
                if (has_e && j != nd - 1) {   // node nd is P_{i+1} of panel i = nd - 1: -d/dd2
                    const double c = ge.tx * gj.tx + ge.ty * gj.ty, s = ge.tx * gj.ty - ge.ty * gj.tx;
                    const double WA = WA0 + wae, WT = WT0 + wte;
                    const double aa = WA * s + WT * c, bb = WA * c - WT * s;
                    ex1 += (aa * dx - bb * dy) * rq;
                    ey1 += (aa * dy + bb * dx) * rq;
                }
            }
            reduce3(ex1, ey1, cphi);
            if (rs == 0 && kn0 <= N) {
                S.gnx[nd] += kInv2Pi * ex1;
                S.gny[nd] += kInv2Pi * ey1;
                if (has_s) {   // dF/dphi_nd from the column of panel nd
                    const double f = -kInv2Pi * cphi / gs.L;
                    S.ghx[nd] += -f * gs.ty;
                    S.ghy[nd] += f * gs.tx;
                }
            }
        }
        __syncthreads();
    }
    if (info && tid == 0) info[b] = conv ? 0 : -2;

    // ---- node gradients: midpoints split evenly, panel vectors P_{i+1} - P_i
    for (int nd = tid; nd <= N; nd += TB) {
        double gx = S.gnx[nd], gy = S.gny[nd];
        if (nd >= 1) {
            gx += 0.5 * S.gmx[nd - 1] + S.ghx[nd - 1];
            gy += 0.5 * S.gmy[nd - 1] + S.ghy[nd - 1];
        }
        if (nd < N) {
            gx += 0.5 * S.gmx[nd] - S.ghx[nd];
            gy += 0.5 * S.gmy[nd] - S.ghy[nd];
        }
        out[2 * nd] = gx;
        out[2 * nd + 1] = gy;
    }
}

template <int TB, int NM>
void launch(const WsView &v, int32_t B, int32_t mixed, const double *xy, const double *dcl, const double *dcp,
            double *dxy, int32_t *info, hipStream_t s) {
    if (mixed)
        adjoint_hs_kernel<float, TB, NM><<<B, TB, 0, s>>>(v, xy, dcl, dcp, dxy, info);
    else
        adjoint_hs_kernel<double, TB, NM><<<B, TB, 0, s>>>(v, xy, dcl, dcp, dxy, info);
}

}  // namespace

hipError_t launch_adjoint_hs(const WsView &v, int32_t B, int32_t max_n1, int32_t mixed, const double *xy,
                             const double *dcl, const double *dcp, double *dxy, int32_t *info, hipStream_t stream) {
    // eight wavefronts per airfoil, two airfoils per CU, as long as the
    // vectors leave room for both
    if (max_n1 <= PANEL_WAVE_MAX_N1)
        launch<512, PANEL_WAVE_MAX_N1>(v, B, mixed, xy, dcl, dcp, dxy, info, stream);
    else
        launch<512, PANEL_NMAX + 1>(v, B, mixed, xy, dcl, dcp, dxy, info, stream);
    return hipGetLastError();
}

}  // namespace panel
