// adjoint.hip -- reverse-mode sensitivity of the lift to the node coordinates
// on gfx950 (the paper optimises airfoil shapes, Sec. 2; this gives the
// shape gradient of the Kutta-Joukowski lift of its panel system).
//
// For one airfoil with solutions x_k of M x_k = r_k (angles k < K) and lift
// Cl_k = -2 sum_i x_k,i L_i / (vinf c), the cotangents dcl_k give
//   xbar   = sum_k dcl_k x_k
//   lambda = M^{-T} w,   w_i = -2 L_i / (vinf c) (i < N),  w_N = 0
//   dP     = -2/(vinf c) sum_i xbar_i dL_i/dP                 (explicit)
//          + sum_j lambda_j sum_k dcl_k dr_k,j/dP              (right-hand side)
//          - sum_{j,i} lambda_j xbar_i dG_ji/dP                (matrix)
// One transposed solve serves all K angles.  It reuses the factors left by
// the forward solve (FP64, or FP32 factors with FP64 refinement of the
// transposed system).  The matrix term re-evaluates closed-form derivatives
// of the panel integral G_ji(m, A, B) (control point m = m_j, panel i from A
// to B, unit tangent t, normal n = (t_y, -t_x), xi = (m-A).t, eta = (m-A).n,
// l1 = log|m-A|^2, l2 = log|m-B|^2, th = angle subtended by the panel):
//   dG/dm = -(1/2pi) [ (l1-l2)/2 t - th n ]
//   dG/dB = I/(2 pi L) + (G/L) t,
//     I = (xi (l1-l2)/2 - L - eta th) t + (-xi th - eta (l1-l2)/2) n
//   dG/dA = -dG/dm - dG/dB                  (translation invariance)
// and, on the diagonal, G_ii = (L/2pi)(1 - log(L/2)), dG_ii/dL = -log(L/2)/2pi.
//
// One workgroup per airfoil.  The transposed solve is adjoint_impl.hpp's.  The
// pairs are evaluated once each, a wavefront per 64 control points (a lane
// each) and a range of panels: the logarithm of |m_j - P_{i+1}|^2 is shared
// with the next panel, the control-point terms stay in the lane, and the four
// panel sums are reduced over the wavefront by a packed butterfly.  In phase f
// wavefront w takes the block w + f (mod the number of blocks) of control
// points against its own panels, so every sum has one writer at a time and a
// fixed order.
//
// What bounds it: FP64 vector arithmetic in the pairs, the serial chain of the
// diagonal blocks in the transposed solve.  Measured against one evaluation
// per control point and another per panel, with a lane per (strided) column
// in the solve (HIP events): 5.48 -> 1.90 ms for 256 sections of order 1025,
// 0.78 -> 0.54 ms for 1024 of order 257 (against one wavefront per section).
#include "adjoint_impl.hpp"

namespace panel {
namespace {

using namespace adj;

constexpr double kInv2Pi = 0.15915494309189535;
constexpr double kInv4Pi = 0.07957747154594767;

template <typename T, int TB, int NM> struct AdjLds {
    double sx[NM + 1], sy[NM + 1];
    double xbar[NM], lam[NM], tmp[NM];
    union {
        SolveLds<T, TB> solve;
        struct {
            double gm[2][NM];     // sums over the panels, per control point
            double ps[NM][4];     // sums over the control points, per panel
        };
    };
    LambdaLds<T, NM> lx;
    double red[3][TB / 64];
    double at[fm::kAtanTab];
    unsigned short perm[NM];
};

// Sums of four values over the wavefront: lane l gets the sum of value l & 3.
// Two packed exchanges leave one value per lane, then the lanes of the same
// value are added up.
__device__ __forceinline__ double wave_sum4(double a, double b, double c, double d) {
    const int lane = threadIdx.x & 63;
    const bool o1 = lane & 1, o2 = lane & 2;
    double ab = (o1 ? b : a) + dpp_d<0xB1>(o1 ? a : b);
    double cd = (o1 ? d : c) + dpp_d<0xB1>(o1 ? c : d);
    double v = (o2 ? cd : ab) + dpp_d<0x4E>(o2 ? ab : cd);
    v += dpp_d<0x124>(v);   // row_ror:4
    v += dpp_d<0x128>(v);   // row_ror:8
    unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    auto l2 = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    auto h2 = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double((int)h2[0], (int)l2[0]) + __hiloint2double((int)h2[1], (int)l2[1]);
}

template <typename T, int TB, int NM>
__global__ __launch_bounds__(TB, TB >= 512 ? 4 : 3) void adjoint_kernel(WsView v, int32_t first, const double *__restrict__ xy,
                                                        const double *__restrict__ dcl,
                                                        const double *__restrict__ dcp, int32_t ka,
                                                        double *__restrict__ dxy, int32_t *__restrict__ info) {
    constexpr int W = TB / 64;
    const int b = v.order[first + blockIdx.x];
    const AirfoilMeta mt = v.meta[b];
    const int N = mt.N, n1 = mt.n1, K = mt.K;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *out = dxy + 2 * (size_t)mt.node_off;
    if (ka >= K) return;   // per-angle pass past this airfoil's angles
    if (v.flag[b] != 0 || n1 > NM) {
        for (int k = tid; k < 2 * (N + 1); k += TB) out[k] = __builtin_nan("");
        if (info && tid == 0) info[b] = v.flag[b] != 0 ? v.flag[b] : -3;
        return;
    }
    __shared__ AdjLds<T, TB, NM> S;
    load_atan_table(S.at);
    const double *P = xy + 2 * (size_t)mt.node_off;
    for (int k = tid; k <= N; k += TB) {
        S.sx[k] = P[2 * k];
        S.sy[k] = P[2 * k + 1];
    }
    const double vinf = v.hdr->vinf, chord = v.chord[b];
    const double *X = v.x + mt.x_off;
    // Cotangent seeds: all angles at once with cl cotangents only (ka < 0,
    // one transposed solve; xbar = sum_k dcl_k x_k), or one angle with its
    // cl and cp cotangents (ka >= 0; xbar = x_ka, the explicit length term
    // scaled by dcl_ka).
    double Sa = 0.0, Ca = 0.0, escale = 1.0;
    if (ka < 0) {
        for (int k = 0; k < K; ++k) {
            const double a = v.alpha[mt.alpha_off + k], d = dcl[mt.alpha_off + k];
            Sa += d * sin(a);
            Ca += d * cos(a);
        }
    } else {
        const double a = v.alpha[mt.alpha_off + ka];
        Sa = sin(a);
        Ca = cos(a);
        escale = dcl[mt.alpha_off + ka];
    }
    const double *cpbar = (ka >= 0 && dcp) ? dcp + mt.s_off + (size_t)ka * N : nullptr;
    const double cpf = -2.0 / (vinf * vinf);
    for (int i = tid; i < n1; i += TB) {
        double s = 0.0;
        if (ka < 0) {
            for (int k = 0; k < K; ++k) s += dcl[mt.alpha_off + k] * X[(size_t)k * n1 + i];
        } else {
            s = X[(size_t)ka * n1 + i];
        }
        S.xbar[i] = s;
    }
    perm_of_pivots(v.piv + mt.piv_off, n1, TB, S.perm);
    const double wscale = -2.0 / (vinf * chord);
    for (int i = tid; i < n1; i += TB) {
        double w = 0.0;
        if (i < N) {
            const double hx = S.sx[i + 1] - S.sx[i], hy = S.sy[i + 1] - S.sy[i];
            w = escale * wscale * sqrt(hx * hx + hy * hy);
            if (cpbar) w += cpbar[i] * cpf * S.xbar[i];
        }
        S.tmp[i] = w;
    }
    __syncthreads();

    const bool conv = solve_lambda<T, TB, NM>(v, mt, S.perm, S.lam, S.tmp, S.solve, S.lx, S.red);
    // info: 0, or -2 when the FP64 refinement of lambda ran out of sweeps
    // (a later per-angle pass never clears an earlier failure)
    if (info && tid == 0) {
        if (!conv) info[b] = -2;
        else if (ka <= 0) info[b] = 0;
    }
    const PanelGeom *geo = v.geom + mt.panel_off;
    for (int i = tid; i < N; i += TB) {
        S.tmp[i] = 1.0 / geo[i].L;   // (tmp is free once lambda is known)
        S.gm[0][i] = S.gm[1][i] = 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e) S.ps[i][e] = 0.0;
    }
    __syncthreads();

    // ---- the panel pairs ---------------------------------------------------
    const int njb = (N + 63) / 64;              // blocks of control points
    const int wa = min(W, njb);                 // wavefronts at work
    const int per = (N + wa - 1) / wa;          // panels of each
    const int i0 = min(per * wave, N), i1 = wave < wa ? min(i0 + per, N) : i0;
    for (int f = 0; f < njb; ++f) {
        if (i0 < i1) {
            int jb = wave + f;
            if (jb >= njb) jb -= njb;
            const int j = 64 * jb + lane, jc = min(j, N - 1);
            const double mx = 0.5 * (S.sx[jc] + S.sx[jc + 1]), my = 0.5 * (S.sy[jc] + S.sy[jc + 1]);
            const double lj = j < N ? S.lam[jc] : 0.0;
            double ax = 0.0, ay = 0.0;
            double Ax = S.sx[i0], Ay = S.sy[i0];
            double d1x = mx - Ax, d1y = my - Ay;
            double l1 = plog(d1x * d1x + d1y * d1y);
            for (int i = i0; i < i1; ++i) {
                const double Bx = S.sx[i + 1], By = S.sy[i + 1];
                const double hx = Bx - Ax, hy = By - Ay;
                const PanelGeom g = geo[i];
                const double L = g.L, iL = S.tmp[i], tx = g.tx, ty = g.ty, nx = ty, ny = -tx;
                const double xb = S.xbar[i];
                const double e2x = mx - Bx, e2y = my - By;
                const double l2 = plog(e2x * e2x + e2y * e2y);
                const double cr = d1x * e2y - d1y * e2x;
                const double th = patan2(cr, d1x * e2x + d1y * e2y, S.at);
                const double hl = 0.5 * (l1 - l2);
                const double xi = d1x * tx + d1y * ty, eta = d1x * nx + d1y * ny;
                const double G = -kInv4Pi * iL *
                                 ((d1x * hx + d1y * hy) * l1 - (e2x * hx + e2y * hy) * l2 - 2.0 * L * L + 2.0 * cr * th);
                double fx = hl * tx - th * nx, fy = hl * ty - th * ny;   // -2pi dG/dm
                const double itt = xi * hl - L - eta * th, inn = -xi * th - eta * hl;
                double bgx = kInv2Pi * iL * (itt * tx + inn * nx) + G * iL * tx;
                double bgy = kInv2Pi * iL * (itt * ty + inn * ny) + G * iL * ty;
                if (i >= 64 * jb && i < 64 * jb + 64) {
                    // the diagonal (j == i): G_ii depends on the panel length
                    // only, dG/dB = dG/dL t, no control-point term
                    const bool dg = j == i;
                    const double dGdL = -kInv2Pi * plog(0.5 * L);
                    bgx = dg ? dGdL * tx : bgx;
                    bgy = dg ? dGdL * ty : bgy;
                    fx = dg ? 0.0 : fx;
                    fy = dg ? 0.0 : fy;
                }
                ax += xb * fx;
                ay += xb * fy;
                const double lk = -kInv2Pi * lj;
                const double s = wave_sum4(lj * bgx, lj * bgy, lk * fx, lk * fy);
                if (lane < 4) __hip_atomic_fetch_add(&S.ps[i][lane], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                d1x = e2x;
                d1y = e2y;
                l1 = l2;
                Ax = Bx;
                Ay = By;
            }
            if (j < N) {   // this phase's only writer of block jb
                S.gm[0][j] += ax;
                S.gm[1][j] += ay;
            }
        }
        __syncthreads();
    }

    // ---- node gradients ------------------------------------------------------
    // control point i sits on panel i (nodes i and i + 1), each node gets half
    // of its m-derivative terms; off the diagonal dA = -dm - dB (the diagonal
    // contributed to dB only, and dA = -dB for it)
    for (int k = tid; k <= N; k += TB) {
        double gx = 0.0, gy = 0.0;
#pragma unroll
        for (int side = 0; side < 2; ++side) {   // panel k - 1 ends, panel k starts at node k
            const int i = k - 1 + side;
            if (i < 0 || i >= N) continue;
            const PanelGeom g = geo[i];
            const double xb = S.xbar[i], li = S.lam[i];
            const double e = escale * wscale * xb;
            const double gmx = -kInv2Pi * li * S.gm[0][i], gmy = -kInv2Pi * li * S.gm[1][i];
            gx += 0.5 * (li * vinf * Sa - gmx);
            gy += 0.5 * (-li * vinf * Ca - gmy);
            if (side == 0) {
                gx += e * g.tx - xb * S.ps[i][0];
                gy += e * g.ty - xb * S.ps[i][1];
            } else {
                gx += -e * g.tx + xb * (S.ps[i][2] + S.ps[i][0]);
                gy += -e * g.ty + xb * (S.ps[i][3] + S.ps[i][1]);
            }
        }
        if (ka <= 0) {   // the first pass writes, later per-angle passes add
            out[2 * k] = gx;
            out[2 * k + 1] = gy;
        } else {
            out[2 * k] += gx;
            out[2 * k + 1] += gy;
        }
    }
}

template <int TB, int NM>
void launch_stream(const WsView &v, int32_t first, int32_t count, int32_t mixed, const double *xy, const double *dcl,
                   const double *dcp, int32_t ka, double *dxy, int32_t *info, hipStream_t s) {
    if (mixed)
        adjoint_kernel<float, TB, NM><<<count, TB, 0, s>>>(v, first, xy, dcl, dcp, ka, dxy, info);
    else
        adjoint_kernel<double, TB, NM><<<count, TB, 0, s>>>(v, first, xy, dcl, dcp, ka, dxy, info);
}

}  // namespace

hipError_t launch_adjoint(const WsView &v, int32_t B, int32_t n_block, int32_t max_n1_block, int32_t max_n1_small,
                          int32_t max_k, int32_t mixed, const double *xy, const double *dcl, const double *dcp, double *dxy,
                          int32_t *info, hipStream_t stream) {
    // without cp cotangents one pass serves all angles; with them one pass
    // per angle index (airfoils with fewer angles skip the later passes)
    const int npass = dcp ? max_k : 1;
    for (int p = 0; p < npass; ++p) {
        const int ka = dcp ? p : -1;
        if (n_block > 0) {
            if (max_n1_block > 512)
                launch_stream<1024, PANEL_NMAX + 1>(v, 0, n_block, mixed, xy, dcl, dcp, ka, dxy, info, stream);
            else
                launch_stream<512, 512>(v, 0, n_block, mixed, xy, dcl, dcp, ka, dxy, info, stream);
        }
        if (B > n_block) {
            // a wavefront each (adjoint_wave.hip) only where short sections
            // leave a workgroup little to share and there are enough of them
            // to fill the GPU.  Wavefronts / workgroups, us, cl cotangents, by
            // sections per CU: FP64, order 65: 138 / 130 at five, 149 / 185 at
            // seven; order 144: 468 / 425 at six, 503 / 491 at seven, 535 / 550
            // at eight.  FP32 factors, order 80: 338 / 330 at six, 388 / 400 at
            // eight; order 97: 913 / 888 at sixteen.  The refinement of lambda
            // leaves workgroups on the shortest systems idle sooner: FP32, order
            // 25: 62 / 62 at four, 75 / 91 at five; order 49: 112 / 96 at four,
            // 138 / 148 at five; order 65: 221 / 223 at five.
            const int32_t per_cu = mixed && max_n1_small <= 56 ? 4 : 6;
            if (B - n_block > per_cu * device_cus() &&
                max_n1_small <= (mixed ? ADJOINT_WAVE_MAX_F32 : ADJOINT_WAVE_MAX_F64)) {
                const hipError_t e =
                    launch_adjoint_wave(v, n_block, B - n_block, mixed, xy, dcl, dcp, ka, dxy, info, stream);
                if (e != hipSuccess) return e;
            } else {
                launch_stream<256, PANEL_WAVE_MAX_N1>(v, n_block, B - n_block, mixed, xy, dcl, dcp, ka, dxy, info,
                                                      stream);
            }
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace panel
