// Instantiations and launches of the row-marching Harris-chain kernels.
#include "rowfuse.h"

namespace fz {

// Zero the arrival counters and every clip's point count (a kernel, so that the
// reset is an ordinary kernel node when the batch is captured into a graph).
__global__ void k_batch_reset(BatchParams bp)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < bp.n_counters) bp.counters[i] = 0u;
    if (i < bp.n_clips && bp.clip[i].count != nullptr) *bp.clip[i].count = 0u;
}

__global__ void k_zero_words(uint32_t* p, int n, uint32_t* count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
    if (i == 0 && count != nullptr) *count = 0u;
}
hipError_t zero_words(uint32_t* p, int n, uint32_t* count, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_words, dim3(std::max(1, (n + 255) / 256)), dim3(256), 0, s, p, n, count);
    return hipGetLastError();
}

hipError_t launch_rowfuse(const RowParams& rp, int K, bool rgb, bool diff, hipStream_t s)
{
    return pick_rowfuse<true>(rp, K, rgb, diff, s);
}

template <bool RGB, bool DIFF>
static hipError_t go_batch(const BatchParams& bp, int blocks, hipStream_t s)
{
    const size_t lds = DIFF ? (size_t)ROW_WAVES * row_mask_bytes(2, bp.max_band) : 0;
    const int n = std::max(bp.n_counters, bp.n_clips);
    hipLaunchKernelGGL(k_batch_reset, dim3((n + 255) / 256), dim3(256), 0, s, bp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = allow_row_lds((const void*)k_rowfuse_batch<2, RGB, DIFF>, lds)) != hipSuccess) return e;
    hipLaunchKernelGGL((k_rowfuse_batch<2, RGB, DIFF>), dim3(blocks), dim3(ROW_WAVES * 64), lds, s, bp);
    return hipGetLastError();
}

hipError_t launch_rowfuse_batch(const BatchParams& bp, bool rgb, bool diff, int blocks, hipStream_t s)
{
    if (rgb) return diff ? go_batch<true, true>(bp, blocks, s) : go_batch<true, false>(bp, blocks, s);
    return diff ? go_batch<false, true>(bp, blocks, s) : go_batch<false, false>(bp, blocks, s);
}

}  // namespace fz
