// refine_block.hip -- kernels that refine one airfoil's FP32 solutions per
// workgroup (refine_block_impl.hpp).
#include "refine_block_impl.hpp"

namespace panel {
namespace {

// Airfoils with fewer than kmin right-hand sides are left to another kernel.
template <int TB, int KG, int NM>
__global__ __launch_bounds__(TB, 2) void refine_kernel(WsView v, int32_t first, int32_t kmin,
                                                       int32_t *__restrict__ info, double tol, int max_iter) {
    __shared__ rfb::WgRefLds<TB, KG, NM> S;
    const int b = v.order[first + blockIdx.x];
    if (v.meta[b].K < kmin) return;
    rfb::wg_refine<TB, KG, NM>(v, b, info, tol, max_iter, S);
}

template <int TB, int NM>
void launch(const WsView &v, int32_t first, int32_t count, int32_t kmin, int32_t max_k, int32_t *info,
            double tol, int32_t max_iter, hipStream_t s) {
    if (max_k > 4)
        refine_kernel<TB, 8, NM><<<count, TB, 0, s>>>(v, first, kmin, info, tol, max_iter);
    else
        refine_kernel<TB, 4, NM><<<count, TB, 0, s>>>(v, first, kmin, info, tol, max_iter);
}

}  // namespace

hipError_t launch_refine_block(const WsView &v, int32_t first, int32_t count, int32_t kmin,
                               int32_t max_n1, int32_t max_k, int32_t waves, int32_t *info, double tol,
                               int32_t max_iter, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    if (waves == 8)
        launch<512, PANEL_NMAX + 1>(v, first, count, kmin, max_k, info, tol, max_iter, stream);
    else if (max_n1 <= PANEL_WAVE_MAX_N1)
        launch<256, PANEL_WAVE_MAX_N1>(v, first, count, kmin, max_k, info, tol, max_iter, stream);
    else   // (four right-hand sides per pass: two workgroups share a CU's LDS)
        refine_kernel<256, 4, 768><<<count, 256, 0, stream>>>(v, first, kmin, info, tol, max_iter);
    return hipGetLastError();
}

}  // namespace panel
