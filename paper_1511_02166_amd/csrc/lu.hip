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
// batch has at most one airfoil per CU (256 systems of order 257: 441 -> 430 us
// in FP64; with more airfoils than CUs, four per airfoil and two airfoils per
// CU keep more systems in flight: 512 of order 257 608 us against 877), and
// always for systems of more than 768 rows.
bool eight_waves(int32_t n_block, int32_t max_n1, int32_t wg_waves) {
    if (max_n1 > 3 * TPB) return true;
    if (wg_waves == 4) return false;
    if (wg_waves == 8) return true;
    return n_block <= device_cus();
}

// Systems within the wave limit by a workgroup each instead of a wavefront
// each.  A wavefront alone on its SIMD takes as long for one system as for a
// thousand, so below about one and a half systems of the largest order per CU
// (FP64; three in FP32, whose matrix cores are faster) the workgroups win.
// Factor + solve, wavefronts against workgroups: FP64, one system of order
// 161 (nine angles) 417 -> 236 us, 256 of order 129 204 -> 187 us, of 257
// 653 -> 441 us, 680 of 66 to 320 next to 320 larger ones 3.13 -> 1.97 ms,
// but 512 of order 129 220 -> 237 us and 256 of order 65 84 -> 91 us; with
// FP32 refinement, 512 of order 129 321 -> 289 us, 1024 436 -> 550 us.
bool small_in_blocks(int32_t max_n1_small, double small_eff, int32_t mixed) {
    if (max_n1_small <= (mixed ? 64 : 96)) return false;
    return small_eff <= (mixed ? 3.0 : 1.5) * device_cus();
}

}  // namespace

hipError_t launch_factor_solve(const WsView &v, int32_t B, int32_t n_block, int32_t max_n1_block,
                               int32_t max_n1_small, double small_eff, int32_t max_k, int32_t mixed, double tol,
                               int32_t max_iter, int32_t *info, int32_t persistent, int32_t wg_waves, hipStream_t stream) {
    hipError_t e = hipSuccess;
    if (persistent && (n_block == 0 || !eight_waves(n_block, max_n1_block, wg_waves == 0 ? 4 : wg_waves))) {
        const int n_small = B - n_block;
        const int grid = std::min(2 * device_cus(), n_block + (n_small + TPB / 64 - 1) / (TPB / 64));
        return launch_lu_batch(v, grid, B, n_block, mixed, tol, max_iter, info, stream);
    }
    const int32_t waves = eight_waves(n_block, max_n1_block, wg_waves) ? 8 : 4;
    if (wg_waves == 0 && small_in_blocks(max_n1_small, small_eff, mixed)) {
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
        // Small systems: a workgroup each where it reads the matrix for
        // several right-hand sides (2048 systems of order 201, four angles:
        // 1.96 -> 0.99 ms) or where the batch leaves most SIMDs idle (256 of
        // order 129: 84 -> 60 us, 512: 46 -> 41, but 1024: 106 -> 170); a
        // wavefront each otherwise, and where the tiling fixes the
        // workgroups.
        const int32_t n_small = B - n_block;
        const int32_t kw = wg_waves != 0 ? PANEL_KMAX : n_small <= 2 * device_cus() ? 0 : 1;
        if (max_k > kw) {
            e = launch_refine_block(v, n_block, n_small, kw + 1, PANEL_WAVE_MAX_N1, max_k, 4, info, tol,
                                    max_iter, stream);
            if (e != hipSuccess) return e;
        }
        if (kw > 0) e = launch_refine_wave(v, n_block, n_small, kw, info, tol, max_iter, stream);
    }
    return e;
}

}  // namespace panel
