// lu.hip -- the factorisation + solve of a batch on gfx950: the choice of
// kernels for a batch.
//
// Sec. 3 of the paper: each airfoil needs an LU decomposition of its dense
// system ((2/3)n^3 operations), and many small systems are solved at once.
// Systems up to the plan's wave limit are factored by one wavefront each
// (lu_wave_impl.hpp), larger ones by a workgroup each (lu_block_impl.hpp); in
// mixed precision the FP64 refinement of the FP32 solutions follows.
#include <algorithm>

#include "panel_internal.hpp"

namespace panel {

// Compute units of the current device.
int device_cus() {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int c = 0;
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) c = 256;
        cus[dev] = c;
    }
    return cus[dev];
}

namespace {

constexpr int TPB = 256;   // threads per workgroup by default (4 wavefronts)

// Eight wavefronts per airfoil for the workgroup kernels: by default when the
// batch has at most one airfoil per CU (four / eight wavefronts, 256 systems in
// FP64: order 320 595 / 571 us; at 257 424 / 426 it no longer matters; with more
// airfoils than CUs, four per airfoil and two airfoils per CU keep more systems
// in flight: 512 of order 320 911 / 1159, of 257 622 / 868), and always for
// systems of more than 768 rows.  (Small systems alone in a batch take four.)
bool eight_waves(int32_t n_block, int32_t max_n1, int32_t wg_waves) {
    if (max_n1 > 3 * TPB) return true;
    if (wg_waves == 4) return false;
    if (wg_waves == 8) return true;
    return n_block <= device_cus();
}

// Systems within the wave limit by a workgroup of four wavefronts each instead
// of a wavefront each.  A wavefront alone on its SIMD takes as long for one
// system as for a thousand; two workgroups share a CU.  Factor + solve,
// wavefronts / workgroups, us, n_small systems of one order (FP32: the LU alone
// differs, refinement by wavefronts on both sides):
//   FP64     1/CU     1.5/CU   2/CU     2.5/CU   FP32   1/CU     2/CU     2.5/CU
//   n1 = 97  136/119  141/143  143/148  170/243         177/158  187/173  205/259
//   n1 = 105 139/125  146/149  147/152  176/256         187/170  196/184  218/281
//   n1 = 113 168/141  173/169  178/174  213/288         210/182  218/198  243/301
//   n1 = 129 205/170  212/205  217/211  259/349         262/225  273/245  305/369
//   n1 = 161 282/212  296/261  303/270  316/445         337/271  359/304  411/457
//   n1 = 257 647/424  695/561  725/622  774/991         704/508  859/705  919/1012
//   n1 = 320 953/595  1023/865 1064/911 1163/1446       1024/741 1151/954 1229/1360
// so equal systems stop at what is resident at once.  (At 65 in FP32: 114/110,
// 126/125, 138/187.)  More of them pay only where the orders spread (`spread`:
// their number over the number weighted by (order / largest)^2, small_eff), so
// that short systems fill the gaps behind the long ones, and until the weighted
// number per CU (before the colon) reaches a limit that grows with the order:
//   FP64, 24-104: 1.03: 143/133, 1.35: 143/159;  65-104: 1.48: 146/189;  24-128:
//   1.28: 212/187, 1.61: 216/224;  24-200: 1.50: 406/360, 1.79: 419/444;
//   150-256: 2.01: 770/694, 2.52: 794/791;  200-319: 1.48: 1051/808, 2.64:
//   1255/1196;  24-319: 2.16: 1147/1051, 2.92: 1290/1396;  but 200-256 (spread
//   1.25): 1.75: 752/762, and 260-319 (1.21): 1.81: 1180/1199
//   FP32, 24-104: 1.70: 195/210;  24-128: 1.61: 273/263, 1.93: 279/310;  128-200:
//   1.61: 489/467, 2.14: 554/565;  150-256: 2.52: 920/866;  200-256: 1.75:
//   857/785, 2.49: 937/919;  200-319: 2.64: 1316/1230;  24-319: 2.16: 1243/1132, 2.92: 1401/1415
// (All with one angle.)  Each further angle costs a wavefront more than a
// workgroup, whose back substitution takes all of them in one pass: the limits
// grow with the mean number of angles k (small_rhs), and in FP32 equal systems
// pay too from some k on.  Wavefronts over workgroups, time:
//   FP32, one order, 2.1 to 3/CU: order 97, k = 4, 8, 12: 0.91 1.02 1.09;  129,
//   k = 2, 4, 8: 0.89 0.97 1.11;  193, k = 2, 4, 8: 0.97 1.05 1.11;  289, k = 1, 2,
//   3, 4, 8: 0.96 0.99 1.03 1.06 1.16
//   FP32, orders of a range: 24-104, 1.70: k = 1, 3, 4: 0.92 1.00 1.03;  65-104
//   (spread 1.48), 1.85: k = 4, 8: 0.94 1.05;  65-128, 2.37: k = 2, 3, 4: 0.95 1.00
//   1.04;  100-143, 2.00: k = 2, 4: 0.91 1.00;  24-200, 2.32: k = 1, 2, 3: 0.94 0.97
//   1.01;  200-319, 2.70: k = 1: 1.08
//   FP64: 24-104, 1.35: k = 1, 2, 3, 4: 0.88 0.94 1.00 1.06;  65-104, 1.40: k = 4,
//   6: 0.93 1.02
// (From three systems per CU on wavefronts, though twelve angles of order 257
// would take 1.23 at 3.5; in FP64 the limits above 112 stay those of one angle.)
bool small_in_blocks(int32_t n_small, int32_t max_n1_small, double small_eff, double small_rhs, int32_t mixed) {
    const int32_t n = max_n1_small, cus = device_cus();
    if (n <= (mixed ? 64 : 96)) return false;
    const double per_cu = small_eff / cus, spread = n_small / small_eff;
    if (n_small <= 2 * cus) return mixed || n > 112 || per_cu <= 1.6;
    const double k = small_rhs, more = k - 1.0;
    if (!mixed) {
        if (n > 112) return spread >= 1.4 && per_cu <= (n <= 224 ? 1.5 : 2.25);
        return per_cu <= 1.5 && (spread >= 1.9 ? per_cu <= 1.2 + 0.08 * more : k >= 6.0);
    }
    if (per_cu > 3.0) return false;
    if (k >= (n <= 126 ? 8.0 : n <= 152 ? 5.0 : n <= 272 ? 4.0 : 3.0)) return true;
    if (n <= 112) return spread >= 1.9 && per_cu <= 1.4 + 0.1 * more;
    if (n > 224) return spread >= 1.2 && per_cu <= 2.85 + 0.15 * more;
    if (spread < (k < 3.0 ? 1.4 : 1.2)) return false;
    return per_cu <= (n <= 144 ? 1.6 + 0.15 * more : 2.0 + 0.2 * more);
}

// Fewest right-hand sides for which a workgroup refines a system within the wave
// limit, instead of a wavefront: it reads the matrix once for several of them,
// and a small batch leaves most SIMDs idle.  Wavefronts / workgroups, us (with the
// same LU before them), systems of one order or of a range:
//   one angle, order 25, 33, 49, 129, 257: 0.25/CU 47/45, 60/60, 80/78, 236/226,
//   696/638;  1/CU 48/47, 60/60, 82/81, 262/238, 707/648;  2/CU 50/51, 63/66,
//   87/88, 276/270, 862/802;  2.5/CU 52/68, 70/91, 98/120, 309/354, 921/965
//   two angles, order 33, 65, 89, 97: 4/CU 101/104, 205/204, 262/239, 297/274;
//   6/CU 117/134, 233/260, 299/304, 343/342;  16/CU 230/314, 513/629, 741/752,
//   898/839;  16/CU of orders 25 to 97: 422/512, 25 to 129: 690/654, 66 to 129:
//   908/842 (rms orders 65, 83, 100)
//   three angles, order 25, 33, 49: 8/CU 133/130, 167/167, 225/209;  16/CU
//   236/252, 298/319, 407/399;  16/CU of orders 25 to 97: 548/524
//   four angles, order 25: 16/CU 291/256
// The batch decides as a whole, as the two kernels run one after the other.  A
// line through the batch (two angles above order 88, three above 40, for
// workgroups) / the batch: two angles, orders 25 to 97, 8/CU 332/291, 16/CU
// 489/429; 65 to 101, 6/CU 376/303; 65 to 128, 8/CU 529/454; three angles, orders
// 25 to 112, 8/CU 404/339.  Tilings that fix the workgroups keep the wavefronts.
// Beside airfoils with more angles, those with one go to workgroups as well up to
// two per CU: a launch for them alone costs 2 us where the whole takes 50 to 100.
int32_t refine_kmin(int32_t n_small, int32_t max_n1_small, double small_eff, int32_t max_k, int32_t wg_waves) {
    const int32_t n = max_n1_small, cus = device_cus();
    if (wg_waves != 0) return PANEL_KMAX + 1;
    if (n_small <= cus || (n_small <= 2 * cus && (n > 64 || max_k > 1))) return 1;
    if (n_small <= 4 * cus) return 2;
    const double rms2 = double(n) * n * small_eff / n_small;   // mean square order
    if (rms2 > 92.0 * 92.0 || (rms2 > 80.0 * 80.0 && n > 112)) return 2;
    return n > 40 ? 3 : 4;
}

}  // namespace

hipError_t launch_factor_solve(const WsView &v, int32_t B, int32_t n_block, int32_t max_n1_block,
                               int32_t max_n1_small, double small_eff, double small_rhs, int32_t max_k,
                               int32_t mixed, double tol, int32_t max_iter, int32_t *info, int32_t persistent,
                               int32_t wg_waves, hipStream_t stream) {
    hipError_t e = hipSuccess;
    if (persistent && (n_block == 0 || !eight_waves(n_block, max_n1_block, wg_waves == 0 ? 4 : wg_waves))) {
        const int n_small = B - n_block;
        const int grid = std::min(2 * device_cus(), n_block + (n_small + TPB / 64 - 1) / (TPB / 64));
        return launch_lu_batch(v, grid, B, n_block, mixed, tol, max_iter, info, stream);
    }
    const int32_t waves = eight_waves(n_block, max_n1_block, wg_waves) ? 8 : 4;
    if (wg_waves == 0 && small_in_blocks(B - n_block, max_n1_small, small_eff, small_rhs, mixed)) {
        // every system by a workgroup, in one launch
        e = launch_lu_block(v, B, n_block, n_block > 0 && eight_waves(B, max_n1_block, 0) ? 8 : 4,
                            n_block > 0 ? max_n1_block : max_n1_small, mixed, info, stream);
    } else {
        e = launch_lu_block(v, n_block, n_block, waves, max_n1_block, mixed, info, stream);
        if (e == hipSuccess) e = launch_lu_wave(v, n_block, B - n_block, mixed, info, stream);
    }
    if (e != hipSuccess) return e;
    if (mixed) {
        e = launch_refine_block(v, 0, n_block, 1, max_n1_block, max_k, waves, info, tol, max_iter, stream);
        if (e != hipSuccess) return e;
        const int32_t n_small = B - n_block;
        const int32_t kmin = refine_kmin(n_small, max_n1_small, small_eff, max_k, wg_waves);
        if (max_k >= kmin) {
            e = launch_refine_block(v, n_block, n_small, kmin, PANEL_WAVE_MAX_N1, max_k, 4, info, tol, max_iter,
                                    stream);
            if (e != hipSuccess) return e;
        }
        if (kmin > 1) e = launch_refine_wave(v, n_block, n_small, kmin - 1, info, tol, max_iter, stream);
    }
    return e;
}

}  // namespace panel
