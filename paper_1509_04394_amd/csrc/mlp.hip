// Cost-model network: a 3-layer FP32 perceptron F -> 64 -> 64 -> 1 with ReLU,
// trained on the GPU by the kernels below to predict log kernel time of a fused
// group from its features (the paper's C_i is a predicted execution time,
// Sec. VI, Fig. 5).
//
// Parameter layout (one flat float array, row-major [out][in]):
//   W1[64][F] b1[64] W2[64][64] b2[64] W3[64] b3[1]
// Loss over a batch of N samples: L = (1/N) sum_n (y_n - t_n)^2.
//
// Every reduction runs in a fixed order (per-block partial sums, then a
// second kernel that adds the partials block by block), so gradients are
// deterministic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "fz_internal.h"

namespace fz {

constexpr int MLP_H = 64;        // hidden width
constexpr int MLP_ROWS = 32;     // samples per tile
constexpr int MLP_THREADS = 256;
constexpr int MLP_MAX_BLOCKS = 512;  // two workgroups a CU; more samples: more tiles each
constexpr int MLP_FMAX = 32;     // most features supported

FZ_HD constexpr int mlp_params(int F) { return MLP_H * F + MLP_H + MLP_H * MLP_H + MLP_H + MLP_H + 1; }

struct MlpOffsets {
    int w1, b1, w2, b2, w3, b3;
};
static inline __host__ __device__ MlpOffsets mlp_offsets(int F)
{
    MlpOffsets o;
    o.w1 = 0;
    o.b1 = o.w1 + MLP_H * F;
    o.w2 = o.b1 + MLP_H;
    o.b2 = o.w2 + MLP_H * MLP_H;
    o.w3 = o.b2 + MLP_H;
    o.b3 = o.w3 + MLP_H;
    return o;
}

// One pass over the samples, forward and (TRAIN) backward, on the matrix cores.
//
// A workgroup of four wavefronts takes tiles of MLP_ROWS samples; wavefront w
// owns the hidden units 16w .. 16w+15 of both layers.  The weights it
// multiplies by are loaded once into registers in the operand layout of the
// 16x16x4 FP32 matrix instruction (lane l: k = l / 16, row or column l % 16;
// result register r: row 4 (l / 16) + r, column l % 16).  A result is a
// sum over samples' operand as it stands: with the samples of the
// contraction taken in the order 4 (l / 16) + r, result register r of dz2 (or
// dz1) is the left operand of step r of dz2^T h1 (dz1^T x), so only the
// right operands (h1, x) and the left operands of the layers (x, h1, dz2)
// pass through LDS.  Row pitches 36 and 68 put the 64 lanes of both access
// patterns on 64 different banks.  The weight gradients stay in the matrix
// accumulators over all tiles of a workgroup and are written once.
//
// What bounds it: the chain of five products with a barrier between them
// (latency; the 246 MFLOP of a step of 8192 samples are 1.6 us at the FP32
// matrix rate).  32 samples a tile give 8192 samples 256 workgroups, one a CU.
// Measured, a step of 8192 samples of 20 features with its reduction and Adam:
// 17.1 us; 88.7 us with one multiply-add a lane at a time, operands read from
// LDS, a forward and a backward launch with the activations in between in
// memory, and the partial gradients added by one dependent chain (34 us of it).
constexpr int MLP_XP = 36, MLP_HP = 68;  // LDS row pitches (floats)

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Sum over the 16 lanes of a row (every lane gets it), by rotations within it.
template <int N>
__device__ __forceinline__ float add_rotated(float v)
{
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + N, 0xf, 0xf, true));  // row_ror:N
}
__device__ __forceinline__ float sum16(float v)
{
    return add_rotated<1>(add_rotated<2>(add_rotated<4>(add_rotated<8>(v))));
}

template <bool TRAIN>
__global__ __launch_bounds__(MLP_THREADS) void k_mlp(const float* __restrict__ prm, int F, const float* __restrict__ x,
                                                     const float* __restrict__ tgt, int n, float* __restrict__ y,
                                                     float* __restrict__ part, float* __restrict__ lpart)
{
    constexpr int RT = MLP_ROWS / 16;  // row tiles of a sample tile
    __shared__ float xs[MLP_ROWS][MLP_XP];
    __shared__ float h1s[MLP_ROWS][MLP_HP];
    __shared__ float d2s[MLP_ROWS][MLP_HP];
    __shared__ float yp[MLP_H / 16][MLP_ROWS];  // each wavefront's share of the output layer's sum
    const MlpOffsets o = mlp_offsets(F);
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), q = (tid & 63) >> 4, c = tid & 15;
    const int j = 16 * w + c;  // this lane's hidden unit
    // operands that stay: W1 and W2 for the layers, W2 for dz1, biases, W3
    float w1[MLP_FMAX / 4], w2[16], w2t[16];
#pragma unroll
    for (int k = 0; k < MLP_FMAX / 4; ++k) w1[k] = 4 * k + q < F ? prm[o.w1 + j * F + 4 * k + q] : 0.0f;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        w2[k] = prm[o.w2 + j * MLP_H + 4 * k + q];
        w2t[k] = TRAIN ? prm[o.w2 + (4 * k + q) * MLP_H + j] : 0.0f;
    }
    const float b1 = prm[o.b1 + j], b2 = prm[o.b2 + j], w3 = prm[o.w3 + j], b3 = prm[o.b3];
    const float inv_n = 1.0f / (float)n;
    f32x4 g2[4] = {}, g1[2] = {};  // gW2 rows 16w.., gW1 rows 16w..
    float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, loss = 0.0f;

    const int tiles = (n + MLP_ROWS - 1) / MLP_ROWS;
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int s0 = t * MLP_ROWS;
        // the rows past the last sample have no activations: those of a sample of
        // zeros may be infinite where the real ones are not, and 0 * inf in a
        // gradient sum is NaN
        auto blank = [&](f32x4(&z)[RT]) {
            if (!TRAIN || s0 + MLP_ROWS <= n) return;
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (s0 + 16 * r + 4 * q + e >= n) z[r][e] = 0.0f;
        };
#pragma unroll
        for (int i = tid; i < MLP_ROWS * MLP_FMAX; i += MLP_THREADS) {
            const int s = i / MLP_FMAX, f = i % MLP_FMAX;
            xs[s][f] = (f < F && s0 + s < n) ? x[(size_t)(s0 + s) * F + f] : 0.0f;
        }
        float tg[RT][4];
        if constexpr (TRAIN) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int s = s0 + 16 * r + 4 * q + e;
                    tg[r][e] = s < n ? tgt[s] : 0.0f;
                }
        }
        __syncthreads();
        f32x4 h1[RT], h2[RT];
        // layer 1: h1 = relu(x W1^T + b1)
        // (the row tiles' sums in turn: one's latency hides the other's)
        f32x4 a[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) a[r] = f32x4{b1, b1, b1, b1};
#pragma unroll
        for (int k = 0; k < MLP_FMAX / 4; ++k)
            if (4 * k < F) {
#pragma unroll
                for (int r = 0; r < RT; ++r) a[r] = mfma4(xs[16 * r + c][4 * k + q], w1[k], a[r]);
            }
        blank(a);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                h1[r][e] = a[r][e] > 0.0f ? a[r][e] : 0.0f;
                h1s[16 * r + 4 * q + e][j] = h1[r][e];
            }
        }
        __syncthreads();
        // layer 2 and this wavefront's share of the output layer
#pragma unroll
        for (int r = 0; r < RT; ++r) a[r] = f32x4{b2, b2, b2, b2};
#pragma unroll
        for (int k = 0; k < 16; ++k)
#pragma unroll
            for (int r = 0; r < RT; ++r) a[r] = mfma4(h1s[16 * r + c][4 * k + q], w2[k], a[r]);
        blank(a);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                h2[r][e] = a[r][e] > 0.0f ? a[r][e] : 0.0f;
                const float v = sum16(w3 * h2[r][e]);
                if (c == 0) yp[w][16 * r + 4 * q + e] = v;
            }
        }
        __syncthreads();
        if constexpr (!TRAIN) {
            if (tid < MLP_ROWS && s0 + tid < n) y[s0 + tid] = b3 + ((yp[0][tid] + yp[1][tid]) + (yp[2][tid] + yp[3][tid]));
            __syncthreads();  // the next tile writes yp
        } else {
            f32x4 d2[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int s = 16 * r + 4 * q + e;
                    const float out = b3 + ((yp[0][s] + yp[1][s]) + (yp[2][s] + yp[3][s]));
                    const float res = s0 + s < n ? out - tg[r][e] : 0.0f;
                    const float dy = 2.0f * res * inv_n;
                    loss = __builtin_fmaf(res, res, loss);
                    gb3 += dy;
                    gw3 = __builtin_fmaf(dy, h2[r][e], gw3);
                    d2[r][e] = h2[r][e] > 0.0f ? dy * w3 : 0.0f;
                    gb2 += d2[r][e];
                    d2s[s][j] = d2[r][e];
                }
            __syncthreads();
            // gW2 += dz2^T h1
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int k = 0; k < 4; ++k) g2[k] = mfma4(d2[r][e], h1s[16 * r + 4 * q + e][16 * k + c], g2[k]);
            // dz1 = (dz2 W2) where h1 > 0, then gW1 += dz1^T x
#pragma unroll
            for (int r = 0; r < RT; ++r) a[r] = f32x4{};
#pragma unroll
            for (int k = 0; k < 16; ++k)
#pragma unroll
                for (int r = 0; r < RT; ++r) a[r] = mfma4(d2s[16 * r + c][4 * k + q], w2t[k], a[r]);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d1 = h1[r][e] > 0.0f ? a[r][e] : 0.0f;
                    gb1 += d1;
#pragma unroll
                    for (int k = 0; k < 2; ++k) g1[k] = mfma4(d1, xs[16 * r + 4 * q + e][16 * k + c], g1[k]);
                }
            }
            __syncthreads();  // the next tile writes xs, h1s
        }
    }
    if constexpr (TRAIN) {
        float* g = part + (size_t)blockIdx.x * mlp_params(F);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * w + 4 * q + e;
#pragma unroll
            for (int k = 0; k < 4; ++k) g[o.w2 + row * MLP_H + 16 * k + c] = g2[k][e];
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (16 * k + c < F) g[o.w1 + row * F + 16 * k + c] = g1[k][e];
        }
        // the four lane groups hold different samples
        auto over_q = [](float v) {
            v += __shfl_xor(v, 16);
            return v + __shfl_xor(v, 32);
        };
        gb1 = over_q(gb1);
        gb2 = over_q(gb2);
        gw3 = over_q(gw3);
        gb3 = over_q(gb3);
        loss = over_q(loss);
        if (q == 0) {
            g[o.b1 + j] = gb1;
            g[o.b2 + j] = gb2;
            g[o.w3 + j] = gw3;
        }
        if (tid == 0) {
            g[o.b3] = gb3;
            lpart[blockIdx.x] = loss * inv_n;
        }
    }
}

// grad[p] = sum over workgroups of part[b][p]; loss likewise.  64 parameters a
// workgroup; its MLP_SLICES slices each add every MLP_SLICES-th row in order,
// then slice 0 adds the slices in order: a fixed order, and a dependent chain
// of rows / MLP_SLICES loads instead of one of all rows.
constexpr int MLP_SLICES = 16;
__global__ __launch_bounds__(64 * MLP_SLICES) void k_mlp_reduce(const float* __restrict__ part,
                                                                const float* __restrict__ lpart, int nblocks, int P,
                                                                float* __restrict__ grad, float* __restrict__ loss)
{
    __shared__ float acc[MLP_SLICES][64];
    const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + lane;
    // column P of the table is the loss
    const float* src = p < P ? part + p : lpart;
    const size_t step = p < P ? (size_t)P : 1;
    float v = 0.0f;
    if (p <= P) {
#pragma unroll 8
        for (int b = sl; b < nblocks; b += MLP_SLICES) v += src[(size_t)b * step];
    }
    acc[sl][lane] = v;
    __syncthreads();
    if (sl != 0 || p > P) return;
    v = acc[0][lane];
#pragma unroll
    for (int k = 1; k < MLP_SLICES; ++k) v += acc[k][lane];
    if (p < P)
        grad[p] = v;
    else if (loss)
        *loss = v;
}

__global__ void k_mlp_adam(float* __restrict__ prm, const float* __restrict__ grad, float* __restrict__ m,
                           float* __restrict__ v, int P, float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    const float g = grad[p];
    const float mm = b1 * m[p] + (1.0f - b1) * g;
    const float vv = b2 * v[p] + (1.0f - b2) * g * g;
    m[p] = mm;
    v[p] = vv;
    const float mh = mm / c1, vh = vv / c2;
    prm[p] -= lr * mh / (__builtin_sqrtf(vh) + eps);
}

// Workgroups of a training step: one a tile, two a compute unit at most.
static int mlp_blocks(int n) { return (int)std::min<int64_t>(((int64_t)n + MLP_ROWS - 1) / MLP_ROWS, MLP_MAX_BLOCKS); }

// Workspace of a training step: the workgroups' partial gradients and losses.
static size_t mlp_ws(int F, int n) { return (size_t)mlp_blocks(n) * (mlp_params(F) + 1) * sizeof(float); }

}  // namespace fz

using namespace fz;

extern "C" {

int32_t fz_mlp_param_count(int32_t n_features) { return (n_features > 0 && n_features <= MLP_FMAX) ? mlp_params(n_features) : -1; }

size_t fz_mlp_workspace_bytes(int32_t n_features, int32_t n)
{
    if (n_features <= 0 || n_features > MLP_FMAX || n <= 0) return 0;
    return mlp_ws(n_features, n);
}

fz_status fz_mlp_forward(const float* d_params, int32_t n_features, const float* d_x, int32_t n, float* d_y,
                         void* stream)
{
    if (!d_params || !d_x || !d_y) return fail(FZ_E_INVALID, "fz_mlp_forward: null pointer");
    if (n_features <= 0 || n_features > MLP_FMAX || n <= 0) return fail(FZ_E_INVALID, "fz_mlp_forward: bad size");
    const int nb = std::min((n + MLP_ROWS - 1) / MLP_ROWS, 4 * MLP_MAX_BLOCKS);
    (void)hipGetLastError();  // drop an error latched by earlier, unrelated runtime calls
    hipLaunchKernelGGL(k_mlp<false>, dim3(nb), dim3(MLP_THREADS), 0, (hipStream_t)stream, d_params, n_features, d_x,
                       nullptr, n, d_y, nullptr, nullptr);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FZ_OK : fail(FZ_E_HIP, std::string("mlp forward: ") + hipGetErrorString(e));
}

fz_status fz_mlp_loss_grad(const float* d_params, int32_t n_features, const float* d_x, const float* d_target,
                           int32_t n, float* d_grad, float* d_loss, void* d_ws, size_t ws_bytes, void* stream)
{
    if (!d_params || !d_x || !d_target || !d_grad) return fail(FZ_E_INVALID, "fz_mlp_loss_grad: null pointer");
    if (n_features <= 0 || n_features > MLP_FMAX || n <= 0) return fail(FZ_E_INVALID, "fz_mlp_loss_grad: bad size");
    if (!d_ws || ws_bytes < mlp_ws(n_features, n))
        return fail(FZ_E_WORKSPACE, "fz_mlp_loss_grad: workspace needs " + std::to_string(mlp_ws(n_features, n)));
    hipStream_t s = (hipStream_t)stream;
    (void)hipGetLastError();  // drop an error latched by earlier, unrelated runtime calls
    const int nb = mlp_blocks(n);
    const int P = mlp_params(n_features);
    float* part = (float*)d_ws;
    float* lpart = part + (size_t)nb * P;
    hipLaunchKernelGGL(k_mlp<true>, dim3(nb), dim3(MLP_THREADS), 0, s, d_params, n_features, d_x, d_target, n, nullptr,
                       part, lpart);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((P + 1 + 63) / 64), dim3(64 * MLP_SLICES), 0, s, part, lpart, nb, P, d_grad,
                       d_loss);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FZ_OK : fail(FZ_E_HIP, std::string("mlp loss/grad: ") + hipGetErrorString(e));
}

fz_status fz_mlp_adam_step(float* d_params, const float* d_grad, float* d_m, float* d_v, int32_t n_params,
                           int32_t step, float lr, float beta1, float beta2, float eps, void* stream)
{
    if (!d_params || !d_grad || !d_m || !d_v) return fail(FZ_E_INVALID, "fz_mlp_adam_step: null pointer");
    if (n_params <= 0 || step < 1) return fail(FZ_E_INVALID, "fz_mlp_adam_step: bad size or step");
    const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    (void)hipGetLastError();  // drop an error latched by earlier, unrelated runtime calls
    hipLaunchKernelGGL(k_mlp_adam, dim3((n_params + 255) / 256), dim3(256), 0, (hipStream_t)stream, d_params, d_grad,
                       d_m, d_v, n_params, lr, beta1, beta2, eps, c1, c2);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FZ_OK : fail(FZ_E_HIP, std::string("mlp adam: ") + hipGetErrorString(e));
}

}  // extern "C"
