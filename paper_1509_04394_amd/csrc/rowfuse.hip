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

// Zero n words (the frame-boundary arrival counters) and the point count (null:
// none); a kernel, not a memset, so that it is an ordinary kernel node when a run
// is captured into a graph.
__global__ void k_zero_words(uint32_t* p, int n, uint32_t* count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
    if (i == 0 && count != nullptr) *count = 0u;
}

template <int K, bool RGB, bool DIFF>
static hipError_t go(const RowParams& rp, hipStream_t s)
{
    const int blocks = (rp.g.total + ROW_WAVES - 1) / ROW_WAVES;
    const size_t lds = DIFF ? (size_t)ROW_WAVES * row_mask_bytes(K, rp.g.band_h) : 0;
    const int nb = DIFF && rp.g.xcount != nullptr ? row_boundaries(rp.g.nstrips, rp.g.nbands, rp.g.nchunks) : 0;
    if (nb > 0 || rp.sp.count != nullptr) {
        hipLaunchKernelGGL(k_zero_words, dim3(std::max(1, (nb + 255) / 256)), dim3(256), 0, s, rp.g.xcount, nb,
                           rp.sp.count);
        const hipError_t z = hipGetLastError();
        if (z != hipSuccess) return z;
    }
    const hipError_t e = allow_row_lds((const void*)k_rowfuse<K, RGB, DIFF>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_rowfuse<K, RGB, DIFF>), dim3(blocks), dim3(ROW_WAVES * 64), lds, s, rp);
    return hipGetLastError();
}

hipError_t launch_rowfuse(const RowParams& rp, int K, bool rgb, bool diff, hipStream_t s)
{
    if (K == 2) {
        if (rgb) return diff ? go<2, true, true>(rp, s) : go<2, true, false>(rp, s);
        return diff ? go<2, false, true>(rp, s) : go<2, false, false>(rp, s);
    }
    if (K == 3) {
        if (rgb) return diff ? go<3, true, true>(rp, s) : go<3, true, false>(rp, s);
        return diff ? go<3, false, true>(rp, s) : go<3, false, false>(rp, s);
    }
    return hipErrorInvalidValue;
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
