// lu_block.hip -- kernels that run one workgroup per airfoil over the first
// entries of the plan's order: the factorisation + solve (lu_block_impl.hpp).
#include "lu_block_impl.hpp"

namespace panel {
namespace {

// RMAX: largest number of rows per thread in a panel (n1 <= TB * RMAX).  With
// 256 threads two workgroups share a CU; 512 threads take the whole CU.
template <typename T, int RMAX, int TB>
__global__ __launch_bounds__(TB, 2) void lu_kernel(WsView v, int32_t *__restrict__ info_out) {
    __shared__ blk::BlkLds<T, TB> S;
    blk::blk_lu<T, TB, RMAX>(v, v.order[blockIdx.x], info_out, S);
}

template <typename T>
void launch_lu(const WsView &v, int32_t count, int32_t waves, int32_t *info, hipStream_t s) {
    if (waves == 8)
        lu_kernel<T, 3, 512><<<count, 512, 0, s>>>(v, info);   // n1 <= 1536
    else
        lu_kernel<T, 3, 256><<<count, 256, 0, s>>>(v, info);   // n1 <= 768
}

}  // namespace

hipError_t launch_lu_block(const WsView &v, int32_t count, int32_t waves, int32_t mixed, int32_t *info,
                           hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    if (mixed)
        launch_lu<float>(v, count, waves, info, stream);
    else
        launch_lu<double>(v, count, waves, info, stream);
    return hipGetLastError();
}

}  // namespace panel
