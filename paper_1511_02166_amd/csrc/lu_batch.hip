// lu_batch.hip -- the persistent kernel that factors, solves and refines a
// whole batch in one launch.
#include "lu_block_impl.hpp"
#include "lu_wave_impl.hpp"
#include "panel_internal.hpp"
#include "refine_block_impl.hpp"

namespace panel {
namespace {

constexpr int TPB = 256;   // threads per workgroup by default (4 wavefronts)

// One launch for a whole batch: persistent workgroups of four wavefronts pop
// airfoils from the plan's LPT order.  The first n_block entries (the largest
// systems) are taken by whole workgroups; once those are gone every
// wavefront pops the smaller systems on its own.  With FP32 factors each
// airfoil's FP64 refinement follows its factorisation in the same workgroup
// or wavefront, so the mixed-precision factor/solve is one launch too.
template <typename T> struct BatchWaveLds {
    union {
        wv::WaveLuLds<T> lu;
        wv::WaveRefLds ref;
    } u;
};
template <typename T> union BatchLds {
    blk::BlkLds<T, TPB> lu;
    rfb::WgRefLds<TPB, 4, 768> ref;
    BatchWaveLds<T> wave[TPB / 64];
};

// One item of each kind.  (Kept out of line, with separate register
// allocations, they spilled more: 600-1000 bytes of scratch per function on
// gfx950 against 216-424 for the whole kernel inlined.)
template <typename T>
__device__ __forceinline__ void batch_wg_item(const WsView &v, int b, int32_t *info, int mixed, double tol,
                                           int max_iter, BatchLds<T> &S) {
    blk::blk_lu<T, TPB, 3, sizeof(T) == 8 ? 3 : 4>(v, b, 3 * TPB, info, S.lu);
    __syncthreads();
    if (mixed) {
        rfb::wg_refine<TPB, 4, 768>(v, b, info, tol, max_iter, S.ref);
        __syncthreads();
    }
}

template <typename T>
__device__ __forceinline__ void batch_wave_item(const WsView &v, int b, int32_t *info, int mixed, double tol,
                                             int max_iter, BatchWaveLds<T> &W) {
    wv::wave_lu<T>(v, b, info, W.u.lu);
    wv::wave_sync();
    if (mixed) {
        wv::wave_refine(v, b, info, tol, max_iter, W.u.ref);
        wv::wave_sync();
    }
}

template <typename T>
__global__ __launch_bounds__(TPB, 2) void batch_kernel(WsView v, int32_t n_block, int32_t B, int32_t mixed,
                                                       double tol, int32_t max_iter, int32_t *__restrict__ info) {
    __shared__ BatchLds<T> S;
    __shared__ int s_item;
    int32_t *q = v.queue;
    for (;;) {
        if (threadIdx.x == 0) s_item = atomicAdd(&q[0], 1);
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(s_item);   // uniform: keep it scalar
        __syncthreads();
        if (it >= n_block) break;
        batch_wg_item<T>(v, v.order[it], info, mixed, tol, max_iter, S);
    }
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // this wavefront's LDS area
    for (;;) {
        int it = 0;
        if ((threadIdx.x & 63) == 0) it = atomicAdd(&q[1], 1);
        it = __builtin_amdgcn_readfirstlane(it);   // lane 0's ticket, in a scalar register
        if (it >= B - n_block) break;
        batch_wave_item<T>(v, v.order[n_block + it], info, mixed, tol, max_iter, S.wave[w]);
    }
    // every workgroup counts itself out; the last one leaves the counters at
    // zero for the next launch on this workspace
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&q[2], 1) == (int)gridDim.x - 1) {
            q[0] = 0;
            q[1] = 0;
            q[2] = 0;
            __threadfence();
        }
    }
}

}  // namespace

hipError_t launch_lu_batch(const WsView &v, int32_t grid, int32_t B, int32_t n_block, int32_t mixed, double tol,
                           int32_t max_iter, int32_t *info, hipStream_t stream) {
    if (mixed)
        batch_kernel<float><<<grid, TPB, 0, stream>>>(v, n_block, B, 1, tol, max_iter, info);
    else
        batch_kernel<double><<<grid, TPB, 0, stream>>>(v, n_block, B, 0, tol, max_iter, info);
    return hipGetLastError();
}

}  // namespace panel
