// lu_block.hip -- kernels that run one workgroup per airfoil over the first
// entries of the plan's order: the factorisation + solve (lu_block_impl.hpp).
#include "lu_block_impl.hpp"

namespace panel {
namespace {

// RMAX: largest number of rows per thread in a panel (n1 <= TB * RMAX); NTM:
// column tiles per wavefront in the trailing update; H: 64-column halves of a
// super-panel.  Entries of the order from n_block on are systems within the
// plan's wave limit: a larger one there (an order that does not match the
// plan) is refused here as by the one-wavefront kernels, so that the answer
// does not depend on which of them the batch takes.
template <typename T, int RMAX, int TB, int NTM, int H>
__global__ __launch_bounds__(TB, 2) void lu_kernel(WsView v, int32_t n_block, int32_t *__restrict__ info_out) {
    __shared__ blk::BlkLds<T, TB, H> S;
    static_assert(RMAX * TB >= PANEL_WAVE_MAX_N1, "every instance holds the small systems");
    blk::blk_lu<T, TB, RMAX, NTM, H>(v, v.order[blockIdx.x],
                                     (int)blockIdx.x < n_block ? RMAX * TB : PANEL_WAVE_MAX_N1, info_out, S);
}

template <typename T>
void launch(const WsView &v, int32_t count, int32_t n_block, int32_t waves, int32_t max_n1, int32_t *info,
            hipStream_t s) {
    constexpr int NTM = sizeof(T) == 8 ? 3 : 4;
    // Above 768 rows the trailing blocks' traffic counts: a rank-128 update
    // halves it (256 systems of order 1025, eight angles: 7.98 -> 7.03 ms in
    // FP64, 4.73 -> 4.57 ms in FP32); below, its longer band solves cost more
    // (256 of order 513 in FP64: 1.49 -> 1.65 ms, in FP32 1.00 -> 1.06).  Up to
    // 512 rows an instance of two row slots spills less than one of three (1024
    // of order 401 in FP64: 2.97 -> 2.85 ms).
    if (waves == 8 && max_n1 > 768)
        lu_kernel<T, 3, 512, sizeof(T) == 8 ? 2 : 4, 2><<<count, 512, 0, s>>>(v, n_block, info);   // n1 <= 1536
    else if (waves == 8)
        lu_kernel<T, 2, 512, NTM, 1><<<count, 512, 0, s>>>(v, n_block, info);   // n1 <= 1024
    else if (max_n1 > 512)
        lu_kernel<T, 3, 256, NTM, 1><<<count, 256, 0, s>>>(v, n_block, info);   // n1 <= 768
    else
        lu_kernel<T, 2, 256, NTM, 1><<<count, 256, 0, s>>>(v, n_block, info);   // n1 <= 512
}

}  // namespace

hipError_t launch_lu_block(const WsView &v, int32_t count, int32_t n_block, int32_t waves, int32_t max_n1,
                           int32_t mixed, int32_t *info, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    if (mixed)
        launch<float>(v, count, n_block, waves, max_n1, info, stream);
    else
        launch<double>(v, count, n_block, waves, max_n1, info, stream);
    return hipGetLastError();
}

}  // namespace panel
