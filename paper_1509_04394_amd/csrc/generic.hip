// Generic single-channel chains on the device.
//
// A group with a window stage runs as one LDS tile kernel (Algorithm 1): a
// workgroup loads the input box of its output tile, grown by the group's halo
// (the sums of the window radii, per axis), into LDS once, then runs the
// window stages one after another between two LDS buffers, each over the box
// that the later stages still need, and writes the last stage's tile to global
// memory.  Point stages never get a pass of their own: the ones before the
// first window stage run on the loaded values, the ones after a window stage
// on that stage's results before they are stored.  A group of point stages
// only is one streaming pass.
//
// The stage list and the stencil weights are kernel arguments (GParams); the
// loops over taps are uniform across the workgroup, so the weights are read
// with scalar loads.  Borders replicate per stage: each stage's cells outside
// the frame hold the value of the cell they clamp to.  The arithmetic order is fixed (stencil: row by row,
// each row left to right, fused multiply-adds from 0; window sum: each row
// left to right, rows top to bottom), so every tile shape and every partition
// gives the same bits.
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "fz_internal.h"
#include "generic.h"

namespace fz {

// Blocks are dealt to the 8 XCDs round-robin (block b on XCD b % 8).  Renumber
// them so that each XCD gets a contiguous run of tiles: neighbouring tiles,
// whose input boxes overlap by the halo, then share that XCD's L2.  A
// bijection on [0, nb) for any nb.
__device__ __forceinline__ int xcd_contiguous(int b, int nb)
{
    const int q = nb >> 3, r = nb & 7, xcd = b & 7, slot = b >> 3;
    return (xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q) + slot;
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Quotient and remainder of e by a wavefront-uniform divisor d > 0 without an
// integer divide (which the hardware lacks): a single-precision estimate,
// then one correction step.  Exact for 0 <= e < 2^20 (a box has at most
// 40960 cells), where the estimate is off by at most one.
struct UDiv {
    int d;
    float inv;
    __device__ __forceinline__ explicit UDiv(int dd) : d(dd), inv(1.0f / (float)dd) {}
    __device__ __forceinline__ int quot(int e, int& rem) const
    {
        int q = (int)((float)e * inv);
        int r = e - q * d;
        if (r < 0) {
            --q;
            r += d;
        } else if (r >= d) {
            ++q;
            r -= d;
        }
        rem = r;
        return q;
    }
};

// One point stage on N values: the kind is tested once for all of them.
template <int N>
__device__ __forceinline__ void gpoints(const GStage& s, float (&v)[N])
{
    switch (s.pk) {
    case FZ_POINT_AFFINE:
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = fmaf(s.a, v[k], s.b);
        break;
    case FZ_POINT_ABS:
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = fabsf(v[k]);
        break;
    case FZ_POINT_SQUARE:
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = v[k] * v[k];
        break;
    case FZ_POINT_SQRTABS:
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = sqrtf(fabsf(v[k]));
        break;
    default:
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = fminf(fmaxf(v[k], s.a), s.b);
    }
}

// The kernel arguments in the constant address space they lie in, so that every
// read of the stage list and the weights is a scalar load: through an ordinary
// reference the marching kernel got a copy of the whole block in scratch memory
// (weights read back lane by lane, 130 registers; 1172 us instead of 348
// on 333x251x200 with 66 look-back taps).
typedef const __attribute__((address_space(4))) GParams GParamsK;
typedef const __attribute__((address_space(4))) float* WeightsK;
__device__ __forceinline__ GStage gst(GParamsK& p, int j)
{
    const auto& q = p.st[j];
    GStage s;
    s.kind = q.kind;
    s.rx = q.rx;
    s.ry = q.ry;
    s.rt = q.rt;
    s.pk = q.pk;
    s.a = q.a;
    s.b = q.b;
    s.woff = q.woff;
    s.buf = q.buf;
    s.slots = q.slots;
    return s;
}

// A block of GQ x GR neighbouring cells of a window stage: each input row of
// the block is read once into registers, GQ + 2RX values, and serves every
// output row it belongs to (a window sum's row sums too).  Every cell sums in
// the order fixed above, so the bits do not depend on the block.  GQ = 5: an
// odd count puts the lanes' first cells on distinct LDS banks (a stride
// coprime with their number); the last stage takes 4, one 16-byte store a row.
// A stencil that looks back adds one frame after another, src(tau) the frame
// tau back, tau = 0 .. rt; the loop over frames is inside the choice of the
// radii (outside it the row addresses of every choice were formed before the
// loop, 143 registers instead of 60).  acc starts from zero.
constexpr int GR = 2;
template <bool STENCIL, int RX, int RY, int GQ>
__device__ __forceinline__ void block_frame(const float* src, int RW, int base, WeightsK w, float (&acc)[GR * GQ])
{
#pragma unroll
    for (int v = -RY; v < RY + GR; ++v) {
        float x[GQ + 2 * RX];
        const int r0 = base + v * RW - RX;
#pragma unroll
        for (int q = 0; q < GQ + 2 * RX; ++q) x[q] = src[r0 + q];
        if constexpr (STENCIL) {
#pragma unroll
            for (int r = 0; r < GR; ++r) {
                if (v - r < -RY || v - r > RY) continue;
#pragma unroll
                for (int u = -RX; u <= RX; ++u) {
                    const float wv = w[(v - r + RY) * (2 * RX + 1) + (u + RX)];
#pragma unroll
                    for (int c = 0; c < GQ; ++c) acc[r * GQ + c] = fmaf(wv, x[c + u + RX], acc[r * GQ + c]);
                }
            }
        } else {
            // (a row sum may start from its first term: acc starts from +0, which absorbs a row sum of -0)
            float h[GQ];
#pragma unroll
            for (int c = 0; c < GQ; ++c) {
                h[c] = x[c];
#pragma unroll
                for (int u = 1; u <= 2 * RX; ++u) h[c] = h[c] + x[c + u];
            }
#pragma unroll
            for (int r = 0; r < GR; ++r) {
                if (v - r < -RY || v - r > RY) continue;
#pragma unroll
                for (int c = 0; c < GQ; ++c) acc[r * GQ + c] = acc[r * GQ + c] + h[c];
            }
        }
    }
}
template <bool STENCIL, int RX, int RY, int GQ, class Src>
__device__ __forceinline__ void block_add(Src&& src, int rt, int RW, int base, WeightsK w, float (&acc)[GR * GQ])
{
    block_frame<STENCIL, RX, RY, GQ>(src(0), RW, base, w, acc);
    if constexpr (STENCIL)  // only stencils look back
#pragma unroll 1
        for (int tau = 1; tau <= rt; ++tau)
            block_frame<STENCIL, RX, RY, GQ>(src(tau), RW, base, w + tau * (2 * RX + 1) * (2 * RY + 1), acc);
}
template <bool STENCIL, int RX, int GQ, class Src>
__device__ __forceinline__ void block_ry(int ry, Src&& src, int rt, int RW, int base, WeightsK w,
                                         float (&acc)[GR * GQ])
{
    switch (ry) {
    case 0: block_add<STENCIL, RX, 0, GQ>(src, rt, RW, base, w, acc); break;
    case 1: block_add<STENCIL, RX, 1, GQ>(src, rt, RW, base, w, acc); break;
    case 2: block_add<STENCIL, RX, 2, GQ>(src, rt, RW, base, w, acc); break;
    default: block_add<STENCIL, RX, 3, GQ>(src, rt, RW, base, w, acc); break;
    }
}
template <bool STENCIL, int GQ, class Src>
__device__ __forceinline__ void block_r(int rx, int ry, Src&& src, int rt, int RW, int base, WeightsK w,
                                        float (&acc)[GR * GQ])
{
    switch (rx) {
    case 0: block_ry<STENCIL, 0, GQ>(ry, src, rt, RW, base, w, acc); break;
    case 1: block_ry<STENCIL, 1, GQ>(ry, src, rt, RW, base, w, acc); break;
    case 2: block_ry<STENCIL, 2, GQ>(ry, src, rt, RW, base, w, acc); break;
    default: block_ry<STENCIL, 3, GQ>(ry, src, rt, RW, base, w, acc); break;
    }
}

// A work item's tile: its input box, RW x RH cells from frame position
// (ox, oy) on, and whether it lies inside the frame.
struct GTile {
    int RW, RH, ox, oy;
    bool interior;  // the whole box
    bool vec_in;    // the box's columns, and rows of frames and box allow aligned four-cell loads
    bool vec_out;   // aligned four-cell stores of the tile
};
template <int TW, int TH>
__device__ __forceinline__ GTile gtile(GParamsK& p, int tx, int ty)
{
    GTile g;
    g.RW = TW + 2 * p.hx;
    g.RH = TH + 2 * p.hy;
    g.ox = tx * TW - p.hx;
    g.oy = ty * TH - p.hy;
    const bool across = g.ox >= 0 && g.ox + g.RW <= p.W, w4 = (p.W & 3) == 0;
    g.interior = across && g.oy >= 0 && g.oy + g.RH <= p.H;
    g.vec_in = across && w4 && ((size_t)p.in & (p.in_u8 ? 3 : 15)) == 0;
    g.vec_out = w4 && (tx + 1) * TW <= p.W && ((size_t)p.out & 15) == 0;
    return g;
}

// Four-cell groups of the input box, aligned in the frame: group kd of row ly
// holds the cells lx = 4 kd - shift + q.  Cells outside the frame take the
// cell they clamp to (the replicate border of the group's input).
struct GGroups {
    int shift, nd;  // nd groups a row
    __device__ __forceinline__ GGroups(GParamsK& p, const GTile& g)
        : shift((4 - (p.hx & 3)) & 3), nd((g.RW + shift + 3) >> 2)
    {
    }
};
// Load group kd of row ly of the frame at element offset fbase.
__device__ __forceinline__ void gload4(GParamsK& p, const GTile& g, const GGroups& n, size_t fbase, int ly, int kd,
                                       float (&v)[4])
{
    const size_t rb = fbase + (size_t)clampi(g.oy + ly, 0, p.H - 1) * p.W;
    const int x0 = g.ox - n.shift + 4 * kd;
    if (g.vec_in) {
        if (p.in_u8) {
            const uint32_t q = *(const uint32_t*)((const uint8_t*)p.in + rb + x0);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = (float)((q >> (8 * k)) & 255u);
        } else {
            const float4 q = *(const float4*)((const float*)p.in + rb + x0);
            v[0] = q.x;
            v[1] = q.y;
            v[2] = q.z;
            v[3] = q.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const size_t gi = rb + clampi(x0 + k, 0, p.W - 1);
            v[k] = p.in_u8 ? (float)((const uint8_t*)p.in)[gi] : ((const float*)p.in)[gi];
        }
    }
}

// After a window stage that is not the last, on a tile that leaves the frame:
// the OW x OH cells it computed (first cell bx, by of the box) that lie outside
// the frame become copies of the cell they clamp to, the replicate border of
// this stage's output, so that the next stage reads without clamping.  Only the
// out-of-frame cells are visited: whole rows above and below the frame, then
// the columns left and right of it.
__device__ __forceinline__ void greplicate(GParamsK& p, const GTile& g, float* dst, int bx, int by, int OW, int OH)
{
    const int y0 = clampi(-g.oy - by, 0, OH), y1 = clampi(p.H - g.oy - by, y0, OH);
    const int x0 = clampi(-g.ox - bx, 0, OW), x1 = clampi(p.W - g.ox - bx, x0, OW);
    const int na = (OH - (y1 - y0)) * OW, ncol = x0 + OW - x1, nall = na + (y1 - y0) * ncol;
    const UDiv by_ow(OW), by_nc(ncol > 0 ? ncol : 1);
    for (int e = threadIdx.x; e < nall; e += BLOCK_THREADS) {
        int cx, cy;
        if (e < na) {
            const int r = by_ow.quot(e, cx);
            cy = r < y0 ? r : r - y0 + y1;
        } else {
            int k;
            const int r = by_nc.quot(e - na, k);
            cy = y0 + r;
            cx = k < x0 ? k : k - x0 + x1;
        }
        const int lx = bx + cx, ly = by + cy;
        dst[ly * g.RW + lx] = dst[(clampi(g.oy + ly, 0, p.H - 1) - g.oy) * g.RW + (clampi(g.ox + lx, 0, p.W - 1) - g.ox)];
    }
}

// The cells one window stage computes, with the halo the later stages need.
struct GRegion {
    int OW, OH, bx, by;  // size, and first cell in box coordinates
};

// One window stage over its region, block by block: `window` adds the block
// with first box cell `base` into acc, `trail` runs the stages that follow it
// up to the next window stage, then the cells go to dst (LDS) or, LAST, to the
// frame at element offset fbase.
template <bool LAST, class Window, class Trail>
__device__ __forceinline__ void gstage(GParamsK& p, const GTile& g, const GRegion& R, float* dst, size_t fbase,
                                       Window&& window, Trail&& trail)
{
    constexpr int GQ = LAST ? 4 : 5;
    const int NQ = (R.OW + GQ - 1) / GQ, NR = (R.OH + GR - 1) / GR;
    const UDiv by_nq(NQ);
    for (int e = threadIdx.x; e < NQ * NR; e += BLOCK_THREADS) {
        int qx;
        const int ry = by_nq.quot(e, qx), cx = qx * GQ;
        // the last row of blocks is moved up to end at the region's last row; the
        // rows it shares with the blocks above are theirs.  The last block of a
        // row may read up to GQ - 1 cells past it (the next row or the padding).
        const int cy = min(ry * GR, R.OH - GR), skip = ry * GR - cy;
        const int lx = R.bx + cx, ly = R.by + cy, base = ly * g.RW + lx;
        const int nk = min(GQ, R.OW - cx);
        float acc[GR * GQ];
#pragma unroll
        for (int k = 0; k < GR * GQ; ++k) acc[k] = 0.0f;
        window(base, acc);
        trail(base, skip, nk, acc);
#pragma unroll
        for (int r = 0; r < GR; ++r) {
            if (r < skip) continue;
            if constexpr (LAST) {
                const int gy = g.oy + ly + r, gx = g.ox + lx;  // the tile's cells: never left of or above the frame
                if (gy >= p.H) continue;
                float* o = p.out + fbase + (size_t)gy * p.W + gx;
                if (g.vec_out) {
                    *(float4*)o = make_float4(acc[r * GQ], acc[r * GQ + 1], acc[r * GQ + 2], acc[r * GQ + 3]);
                } else {
#pragma unroll
                    for (int c = 0; c < GQ; ++c)
                        if (gx + c < p.W) o[c] = acc[r * GQ + c];
                }
            } else {
#pragma unroll
                for (int c = 0; c < GQ; ++c)
                    if (c < nk) dst[base + r * g.RW + c] = acc[r * GQ + c];
            }
        }
    }
}

// What bounds it: instruction issue (the stage list is interpreted) and LDS
// reads, (5 + 2r) (2 + 2r) words for ten cells.  Interpreting per block of
// cells instead of per cell, four-cell loads and stores, and border tiles on
// the same path with a replicate pass instead of clamped reads per tap
// took 800x600x64 u8 (3x3 stencil, |x|, 3x3 window sum) from 182 to 96 us and a
// nine-stage f32 chain at 320x240x64 from 360 to 88 us.
template <int TW, int TH>
__global__ __launch_bounds__(BLOCK_THREADS) void k_gtile(const GParams)
{
    GParamsK& p = *(const GParamsK*)__builtin_amdgcn_kernarg_segment_ptr();
    extern __shared__ float glds[];
    int b = xcd_contiguous(blockIdx.x, gridDim.x);
    const int tx = b % p.tiles_x;
    b /= p.tiles_x;
    const GTile g = gtile<TW, TH>(p, tx, b % p.tiles_y);
    const size_t fbase = (size_t)(b / p.tiles_y) * p.W * p.H;
    float* src = glds;
    float* dst = glds + g.RW * g.RH;

    int lead = 0;
    while (lead < p.n && p.st[lead].kind == G_POINT) ++lead;
    const GGroups n(p, g);
    const UDiv by_nd(n.nd);
    for (int e = threadIdx.x; e < n.nd * g.RH; e += BLOCK_THREADS) {
        int kd;
        const int ly = by_nd.quot(e, kd);
        float v[4];
        gload4(p, g, n, fbase, ly, kd, v);
        for (int j = 0; j < lead; ++j) gpoints(gst(p, j), v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int lx = 4 * kd - n.shift + k;
            if (lx >= 0 && lx < g.RW) src[ly * g.RW + lx] = v[k];
        }
    }
    __syncthreads();

    int i = lead, hx = p.hx, hy = p.hy;
    while (true) {
        const GStage s = gst(p, i);
        int j = i + 1;
        while (j < p.n && p.st[j].kind == G_POINT) ++j;
        hx -= s.rx;  // halo still needed after this stage
        hy -= s.ry;
        const GRegion R{TW + 2 * hx, TH + 2 * hy, p.hx - hx, p.hy - hy};
        WeightsK w = p.w + s.woff;
        auto window = [&](int base, auto& acc) {
            constexpr int GQ = sizeof(acc) / sizeof(float) / GR;
            auto frame = [&](int) { return (const float*)src; };
            if (s.kind == G_STENCIL)
                block_r<true, GQ>(s.rx, s.ry, frame, 0, g.RW, base, w, acc);
            else
                block_r<false, GQ>(s.rx, s.ry, frame, 0, g.RW, base, w, acc);
        };
        auto trail = [&](int, int, int, auto& acc) {
            for (int q = i + 1; q < j; ++q) gpoints(gst(p, q), acc);
        };
        if (j == p.n) {
            gstage<true>(p, g, R, nullptr, fbase, window, trail);
            return;
        }
        gstage<false>(p, g, R, dst, 0, window, trail);
        __syncthreads();
        if (!g.interior) {
            greplicate(p, g, dst, R.bx, R.by, R.OW, R.OH);
            __syncthreads();
        }
        float* tmp = src;
        src = dst;
        dst = tmp;
        i = j;
    }
}

// A group of point stages: one pass, each thread groups of four pixels strided
// by the grid (one pixel where the count is no multiple of four or a buffer is
// not aligned).  Bound by memory: 800x600x64 u8 in 29 us (5.3 TB/s; 67 us with
// one pixel a thread), f32 in 39 us (6.3 TB/s; 68 us).
template <int V>
__global__ __launch_bounds__(BLOCK_THREADS) void k_gstream(const GParams p)
{
    const size_t n = (size_t)p.W * p.H * p.T / V;
    const size_t stride = (size_t)gridDim.x * BLOCK_THREADS;
    for (size_t i = (size_t)blockIdx.x * BLOCK_THREADS + threadIdx.x; i < n; i += stride) {
        float v[V];
        if constexpr (V == 4) {
            if (p.in_u8) {
                const uint32_t q = ((const uint32_t*)p.in)[i];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = (float)((q >> (8 * k)) & 255u);
            } else {
                const float4 q = ((const float4*)p.in)[i];
                v[0] = q.x;
                v[1] = q.y;
                v[2] = q.z;
                v[3] = q.w;
            }
        } else {
            v[0] = p.in_u8 ? (float)((const uint8_t*)p.in)[i] : ((const float*)p.in)[i];
        }
        for (int j = 0; j < p.n; ++j) gpoints(p.st[j], v);
        if constexpr (V == 4)
            ((float4*)p.out)[i] = make_float4(v[0], v[1], v[2], v[3]);
        else
            p.out[i] = v[0];
    }
}

// ------------------------------------------------------------ temporal stages
//
// Table II's IIR filter is a point operation over several frames: per pixel,
// y[t] = a x[t] + (1 - a) y[t-1] with y[-1] := x[0].  It runs in double
// precision -- the state and fma(a, x, (1 - a) y_prev), with 1 - a exact in
// double for an f32 a -- and each output is rounded once to f32: in f32 the
// recursion's rounding errors would pile up over about 1/a frames (a = 0.05
// gave 1.1e-4 on a 0-255 scale).  A stencil
// may also look rt frames back (Table I's spatio-temporal class):
// out(t) = sum over tau = 0..rt (this frame first) of the frame t - tau
// window, frames before the first replicating the first; each frame's window
// is summed as the spatial stencil sums it, continuing one fused multiply-add
// chain.  Groups with such stages march through frames in order.

// One IIR step of the cell whose running state is *state (first: frame 0).
__device__ __forceinline__ float giir(const GStage& s, float v, double* state, bool first)
{
    const double a = (double)s.a, x = (double)v;
    const double prev = first ? x : *state;
    const double y = fma(a, x, (1.0 - a) * prev);
    *state = y;
    return (float)y;
}

// A group with a window stage and a temporal stage (an IIR, or a stencil that
// looks back): one workgroup owns an output tile and a run of tt frames and
// marches through frames t0 - ht .. t0 + tt - 1 in order (from frame 0 when the
// run starts within ht frames of it, and always from frame 0 for an IIR, whose
// runs are the whole clip).  Per frame it loads the input box once and runs the
// stages as the tile kernel does; a stencil that looks back reads its earlier
// input frames from a ring in LDS, an IIR keeps its state per box cell in
// LDS (layout: march_layout).  The frames before t0 only fill the rings: a
// stage skips a frame whose ring is not yet full, and nothing is stored before
// t0.  Every stage evaluates exactly as in the tile kernel, so the bits do not
// depend on the partition, the tile or the frame run.  Bound as the tile
// kernel, and by the barriers between a frame's steps; on the tile kernel's
// blocks 333x251x200 with 66 look-back taps went from 878 to 348 us.
template <int TW, int TH>
__global__ __launch_bounds__(BLOCK_THREADS) void k_gmarch(const GParams)
{
    GParamsK& p = *(const GParamsK*)__builtin_amdgcn_kernarg_segment_ptr();
    extern __shared__ float glds[];
    int b = xcd_contiguous(blockIdx.x, gridDim.x);
    const int tx = b % p.tiles_x;
    b /= p.tiles_x;
    const GTile g = gtile<TW, TH>(p, tx, b % p.tiles_y);
    const int CELLS = g.RW * g.RH;
    const int t0 = (b / p.tiles_y) * p.tt;
    const int t1 = min(p.T, t0 + p.tt);
    const int fs = max(0, t0 - p.ht);  // first frame marched
    const size_t P = (size_t)p.W * p.H;

    int lead = 0;
    while (lead < p.n && !g_is_window(p.st[lead].kind)) ++lead;
    const GGroups n(p, g);
    const UDiv by_nd(n.nd);

    if (p.ck_n > 0 && t0 > 0) {
        // the leading IIRs resume from the first pass's state after frame t0 - 1
        const double* ck = p.ckpt + (size_t)(t0 / p.tt - 1) * p.ck_n * P;
        const UDiv by_rw(g.RW);
        for (int e = threadIdx.x; e < CELLS; e += BLOCK_THREADS) {
            int lx;
            const int ly = by_rw.quot(e, lx);
            const size_t gi = (size_t)clampi(g.oy + ly, 0, p.H - 1) * p.W + clampi(g.ox + lx, 0, p.W - 1);
            int k = 0;
            for (int j = 0; j < lead; ++j) {
                const GStage sj = gst(p, j);
                if (sj.kind != G_IIR) continue;
                ((double*)(glds + sj.buf))[e] = ck[(size_t)k * P + gi];
                ++k;
            }
        }
        __syncthreads();
    }

    for (int f = fs; f < t1; ++f) {
        const bool first = f == 0;
        const size_t fbase = (size_t)f * P;
        {
            const GStage s0 = gst(p, lead);
            float* dst = glds + s0.buf + (f % s0.slots) * CELLS;
            for (int e = threadIdx.x; e < n.nd * g.RH; e += BLOCK_THREADS) {
                int kd;
                const int ly = by_nd.quot(e, kd);
                float v[4];
                gload4(p, g, n, fbase, ly, kd, v);
                const int lx = 4 * kd - n.shift, cell = ly * g.RW + lx;
                for (int q = 0; q < lead; ++q) {
                    const GStage sq = gst(p, q);
                    if (sq.kind != G_IIR) {
                        gpoints(sq, v);
                        continue;
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (lx + k >= 0 && lx + k < g.RW)
                            v[k] = giir(sq, v[k], (double*)(glds + sq.buf) + cell + k, first);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (lx + k >= 0 && lx + k < g.RW) dst[cell + k] = v[k];
            }
        }
        __syncthreads();

        int i = lead, hx = p.hx, hy = p.hy, back = 0;
        while (true) {
            const GStage s = gst(p, i);
            int j = i + 1;
            while (j < p.n && !g_is_window(p.st[j].kind)) ++j;
            const bool last = j == p.n;
            back += s.rt;
            hx -= s.rx;
            hy -= s.ry;
            // this stage's input ring holds frames f - rt .. f (replicated before frame 0)
            const bool ready = fs == 0 || f >= fs + back;
            if (ready && (!last || f >= t0)) {
                const GRegion R{TW + 2 * hx, TH + 2 * hy, p.hx - hx, p.hy - hy};
                auto window = [&](int base, auto& acc) {
                    constexpr int GQ = sizeof(acc) / sizeof(float) / GR;
                    auto frame = [&](int tau) {
                        return (const float*)(glds + s.buf + (max(f - tau, 0) % s.slots) * CELLS);
                    };
                    WeightsK w = p.w + s.woff;
                    if (s.kind == G_STENCIL)
                        block_r<true, GQ>(s.rx, s.ry, frame, s.rt, g.RW, base, w, acc);
                    else
                        block_r<false, GQ>(s.rx, s.ry, frame, 0, g.RW, base, w, acc);
                };
                auto trail = [&](int base, int skip, int nk, auto& acc) {
                    constexpr int GQ = sizeof(acc) / sizeof(float) / GR;
                    for (int q = i + 1; q < j; ++q) {
                        const GStage sq = gst(p, q);
                        if (sq.kind != G_IIR) {
                            gpoints(sq, acc);
                            continue;
                        }
                        // a cell's state is stepped once a frame, by the block that owns the cell
#pragma unroll
                        for (int k = 0; k < GR * GQ; ++k)
                            if (k / GQ >= skip && k % GQ < nk)
                                acc[k] = giir(sq, acc[k], (double*)(glds + sq.buf) + base + k / GQ * g.RW + k % GQ, first);
                    }
                };
                if (last) {
                    gstage<true>(p, g, R, nullptr, fbase, window, trail);
                } else {
                    float* dst = glds + p.st[j].buf + (f % p.st[j].slots) * CELLS;
                    gstage<false>(p, g, R, dst, 0, window, trail);
                    if (!g.interior) {
                        __syncthreads();
                        greplicate(p, g, dst, R.bx, R.by, R.OW, R.OH);
                    }
                }
            }
            if (last) break;
            __syncthreads();
            i = j;
        }
        __syncthreads();  // the next frame's load reuses the buffers
    }
}

// A group of point and IIR stages only: each thread owns PX neighbouring
// pixels and marches through every frame in order; D frames are loaded before
// any is processed, so D loads per thread are in flight at once.  With ONE
// (the group has a single IIR) its states are PX registers; otherwise the
// IIR states (doubles) live in LDS, PX per thread and IIR stage (GStage::buf
// is the stage's offset there, in doubles): registers indexed by a stage
// number only known at run time would have gone to scratch memory.
//
// With CKPT, the kernel is the first pass of a checkpointed group: it runs
// the group's leading point and IIR stages only (p.n of them), stores no
// output, and after the last frame of every frame run but the last writes
// each IIR's state to p.ckpt[run][IIR][pixel].
//
// SINGLE (the group is one IIR and nothing else): its coefficient is read once.
// Reading the stage list for every frame, with a scalar load's latency each
// time and two wavefronts a SIMD to hide it, bound the kernel: 800x600x1000 u8
// with a checkpoint every 16 frames took 329 us and takes 161 us.
// Without RAW its input is f32: a test of the type at every load kept the loads
// from being in flight together (192x432x600 f32 333 us; now 147).
template <int PX, int D, bool CKPT, bool ONE, bool RAW = false, bool SINGLE = false>
__global__ __launch_bounds__(BLOCK_THREADS) void k_gstream_t(const GParams p)
{
    static_assert(!SINGLE || ONE, "one IIR: its states in registers");
    extern __shared__ double gstate[];
    double rstate[PX];  // ONE: the IIR's states
#pragma unroll
    for (int k = 0; k < PX; ++k) rstate[k] = 0.0;
    const double a1 = (double)p.st[0].a, b1 = 1.0 - a1;  // SINGLE
    const size_t P = (size_t)p.W * p.H;
    const size_t i0 = ((size_t)blockIdx.x * BLOCK_THREADS + threadIdx.x) * PX;
    if (i0 >= P) return;  // no barrier below
    int next_save = p.tt, saved = 0;  // CKPT: frames until the run's end, runs saved
    for (int t = 0; t < p.T; t += D) {
        // RAW (u8 input, four pixels): the D frames' bytes stay packed, one
        // register per frame, so many frames can be in flight
        float v[RAW ? 1 : D][PX];
        uint32_t raw[RAW ? D : 1];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (t + d >= p.T) break;
            const size_t gi = (size_t)(t + d) * P + i0;
            if constexpr (RAW) {
                raw[d] = *(const uint32_t*)((const uint8_t*)p.in + gi);
            } else if constexpr (PX == 4) {
                if (!SINGLE && p.in_u8) {
                    const uchar4 q = *(const uchar4*)((const uint8_t*)p.in + gi);
                    v[d][0] = q.x;
                    v[d][1] = q.y;
                    v[d][2] = q.z;
                    v[d][3] = q.w;
                } else {
                    const float4 q = *(const float4*)((const float*)p.in + gi);
                    v[d][0] = q.x;
                    v[d][1] = q.y;
                    v[d][2] = q.z;
                    v[d][3] = q.w;
                }
            } else {
                v[d][0] = p.in_u8 ? (float)((const uint8_t*)p.in)[gi] : ((const float*)p.in)[gi];
            }
        }
        if constexpr (SINGLE) {
            if (t == 0) {  // y[-1] := x[0]
#pragma unroll
                for (int k = 0; k < PX; ++k)
                    rstate[k] = RAW ? (double)((raw[0] >> (8 * k)) & 255u) : (double)v[0][k];
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (t + d >= p.T) break;
            float w[PX];
#pragma unroll
            for (int k = 0; k < PX; ++k) w[k] = RAW ? (float)((raw[RAW ? d : 0] >> (8 * k)) & 255u) : v[RAW ? 0 : d][k];
            bool save = false;
            if constexpr (CKPT) {
                save = --next_save == 0;
                if (save) {
                    next_save = p.tt;
                    ++saved;
                    save = t + d + 1 < p.T;
                }
            }
            if constexpr (SINGLE) {
#pragma unroll
                for (int k = 0; k < PX; ++k) {
                    rstate[k] = fma(a1, (double)w[k], b1 * rstate[k]);
                    w[k] = (float)rstate[k];
                }
                if (CKPT && save) {
                    double* ck = (double*)p.ckpt + (size_t)(saved - 1) * P + i0;
#pragma unroll
                    for (int k = 0; k < PX; ++k) ck[k] = rstate[k];
                }
            } else {
                const bool first = t + d == 0;
                int n_iir = 0;
                for (int j = 0; j < p.n; ++j) {
                    const GStage s = p.st[j];
                    if (s.kind == G_IIR) {
                        double* sp = ONE ? rstate : gstate + s.buf + threadIdx.x * PX;
                        const double a = (double)s.a;
#pragma unroll
                        for (int k = 0; k < PX; ++k) {
                            const double x = (double)w[k];
                            const double prev = ONE ? rstate[k] : sp[k];
                            const double y = fma(a, x, (1.0 - a) * (first ? x : prev));
                            if (ONE)
                                rstate[k] = y;
                            else
                                sp[k] = y;
                            w[k] = (float)y;
                        }
                        if (CKPT && save) {
                            double* ck = (double*)p.ckpt + ((size_t)(saved - 1) * p.ck_n + n_iir) * P + i0;
#pragma unroll
                            for (int k = 0; k < PX; ++k) ck[k] = ONE ? rstate[k] : sp[k];
                        }
                        ++n_iir;
                    } else {
                        gpoints(s, w);
                    }
                }
            }
            if constexpr (!CKPT) {
                const size_t gi = (size_t)(t + d) * P + i0;
                if constexpr (PX == 4)
                    *(float4*)(p.out + gi) = make_float4(w[0], w[1], w[2], w[3]);
                else
                    p.out[gi] = w[0];
            }
        }
    }
}

template <typename K>
static hipError_t allow_lds(K kernel, int lds)
{
    if (lds <= 65536) return hipSuccess;
    // dynamic LDS beyond 64 KB (the CU has 160 KB)
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
}

template <int TW, int TH>
static hipError_t launch_tile(const GParams& gp, int lds, bool march, int nchunks, hipStream_t s)
{
    const long long blocks = (long long)gp.tiles_x * gp.tiles_y * (march ? nchunks : gp.T);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipError_t e;
    if (march) {
        if ((e = allow_lds(k_gmarch<TW, TH>, lds)) != hipSuccess) return e;
        k_gmarch<TW, TH><<<dim3((unsigned)blocks), dim3(BLOCK_THREADS), lds, s>>>(gp);
    } else {
        if ((e = allow_lds(k_gtile<TW, TH>, lds)) != hipSuccess) return e;
        k_gtile<TW, TH><<<dim3((unsigned)blocks), dim3(BLOCK_THREADS), lds, s>>>(gp);
    }
    return hipGetLastError();
}

// Launch a group of point and IIR stages through k_gstream_t (the whole group,
// or with CKPT the first pass of a checkpointed group).
template <bool CKPT>
static hipError_t launch_stream_t(GParams gp, const void* in, size_t P, hipStream_t s)
{
    int n_iir = 0;
    for (int j = 0; j < gp.n; ++j) n_iir += gp.st[j].kind == G_IIR ? 1 : 0;
    const bool one = n_iir == 1;
    // four pixels per thread where aligned; with one IIR on u8 input (its
    // states in registers, the input bytes kept packed) 32 frames are loaded
    // ahead: every thread marches all frames in order, so the kernel lives on
    // the bytes in flight, and a pixel per thread (64-byte pieces of frames
    // far apart) read at a fraction of the bandwidth
    const bool vec = P % 4 == 0 && ((uintptr_t)in % (gp.in_u8 ? 4 : 16)) == 0 &&
                     (CKPT || ((uintptr_t)gp.out % 16) == 0);
    const int px = vec ? 4 : 1;
    n_iir = 0;
    for (int j = 0; j < gp.n; ++j)
        if (gp.st[j].kind == G_IIR) gp.st[j].buf = (n_iir++) * BLOCK_THREADS * px;
    const int lds = one ? 0 : n_iir * BLOCK_THREADS * px * 8;  // doubles; a 4-pixel run with 16 IIRs: 128 KB
    hipError_t e = hipSuccess;
    if (lds > 65536) e = vec ? allow_lds(k_gstream_t<4, 8, CKPT, false>, lds) : allow_lds(k_gstream_t<1, 8, CKPT, false>, lds);
    if (e != hipSuccess) return e;
    const size_t threads = P / px;
    const unsigned blocks = (unsigned)((threads + BLOCK_THREADS - 1) / BLOCK_THREADS);
    if (vec && gp.n == 1 && gp.in_u8)
        k_gstream_t<4, 32, CKPT, true, true, true><<<dim3(blocks), dim3(BLOCK_THREADS), 0, s>>>(gp);
    else if (vec && gp.n == 1)
        k_gstream_t<4, 8, CKPT, true, false, true><<<dim3(blocks), dim3(BLOCK_THREADS), 0, s>>>(gp);
    else if (vec && one && gp.in_u8)
        k_gstream_t<4, 32, CKPT, true, true><<<dim3(blocks), dim3(BLOCK_THREADS), lds, s>>>(gp);
    else if (vec && one)
        k_gstream_t<4, 8, CKPT, true><<<dim3(blocks), dim3(BLOCK_THREADS), lds, s>>>(gp);
    else if (vec)
        k_gstream_t<4, 8, CKPT, false><<<dim3(blocks), dim3(BLOCK_THREADS), lds, s>>>(gp);
    else if (one)
        k_gstream_t<1, 8, CKPT, true><<<dim3(blocks), dim3(BLOCK_THREADS), lds, s>>>(gp);
    else
        k_gstream_t<1, 8, CKPT, false><<<dim3(blocks), dim3(BLOCK_THREADS), lds, s>>>(gp);
    return hipGetLastError();
}

size_t ckpt_bytes(const fz_plan& p, const Segment& g)
{
    if (!p.generic || !g.ckpt || g.tpb <= 0) return 0;
    GStage st[G_MAX_STAGES];
    g_stage_list(p.stages.data(), g.first, g.last, st);
    const int n_iir = g_ckpt_iirs(st, g.last - g.first + 1);
    const size_t runs = (size_t)(p.T + g.tpb - 1) / g.tpb;
    return runs > 1 ? (runs - 1) * n_iir * (size_t)p.W * p.H * sizeof(double) : 0;
}

int launch_generic(const fz_plan& p, const Segment& g, const void* in, void* out, void* ckpt, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    GParams gp{};
    gp.in = in;
    gp.out = (float*)out;
    gp.W = p.W;
    gp.H = p.H;
    gp.T = p.T;
    gp.in_u8 = p.stages[g.first].in_dtype == FZ_U8;
    gp.n = g.last - g.first + 1;
    gp.hx = g.halo;
    gp.hy = g.halo_y;
    if (gp.n > G_MAX_STAGES) return hipErrorInvalidValue;
    const int need = g_stage_list(p.stages.data(), g.first, g.last, gp.st);
    if (need > G_MAX_WEIGHTS) return hipErrorInvalidValue;  // the planner never forms such a group
    int nw = 0;
    for (int j = g.first; j <= g.last; ++j) {
        GStage& d = gp.st[j - g.first];
        if (d.kind != G_STENCIL) continue;
        const int cnt = (2 * d.rx + 1) * (2 * d.ry + 1) * (d.rt + 1);
        d.woff = nw;
        std::copy(p.gweights.begin() + p.gwoff[j], p.gweights.begin() + p.gwoff[j] + cnt, gp.w + nw);
        nw += cnt;
    }
    bool has_iir = false;
    const bool temporal = g_temporal(gp.st, gp.n, &has_iir, &gp.ht);
    const size_t P = (size_t)p.W * p.H;
    if (g.engine == FZ_ENGINE_STREAM) {
        if (temporal) return launch_stream_t<false>(gp, in, P, s);  // point and IIR stages, all frames
        const size_t n = P * p.T;
        const bool vec = n % 4 == 0 && ((uintptr_t)in % (gp.in_u8 ? 4 : 16)) == 0 && ((uintptr_t)out % 16) == 0;
        const size_t want = (n / (vec ? 4 : 1) + BLOCK_THREADS - 1) / BLOCK_THREADS;
        const unsigned blocks = (unsigned)std::min<size_t>(want, 256 * 32);
        if (vec)
            k_gstream<4><<<dim3(blocks), dim3(BLOCK_THREADS), 0, s>>>(gp);
        else
            k_gstream<1><<<dim3(blocks), dim3(BLOCK_THREADS), 0, s>>>(gp);
        return hipGetLastError();
    }
    if (g.engine == FZ_ENGINE_JIT && !temporal) return launch_jit(p, g, in, out, nullptr, stream);
    gp.tiles_x = (p.W + g.tile_w - 1) / g.tile_w;
    gp.tiles_y = (p.H + g.tile_h - 1) / g.tile_h;
    int nchunks = 1;
    if (temporal) {
        gp.tt = g.tpb;
        if (gp.tt < 1 || (has_iir && !g.ckpt && gp.tt < p.T)) return hipErrorInvalidValue;
        nchunks = (p.T + gp.tt - 1) / gp.tt;
        if (g.ckpt && nchunks > 1) {
            // first pass: the leading point and IIR stages over every pixel, checkpoints only
            if (!ckpt) return hipErrorInvalidValue;
            gp.ck_n = g_ckpt_iirs(gp.st, gp.n);
            gp.ckpt = (const double*)ckpt;
            GParams g1 = gp;
            int lead = 0;
            while (lead < gp.n && !g_is_window(gp.st[lead].kind)) ++lead;
            g1.n = lead;
            g1.out = nullptr;
            const hipError_t e = launch_stream_t<true>(g1, in, P, s);
            if (e != hipSuccess) return e;
        }
        if (g.engine == FZ_ENGINE_JIT) return launch_jit(p, g, in, out, ckpt, stream);
        const int floats = march_layout(gp.st, gp.n, (g.tile_w + 2 * gp.hx) * (g.tile_h + 2 * gp.hy));
        if ((floats + GEN_PAD) * 4 != g.lds_bytes) return hipErrorInvalidValue;
    }
    switch (g.tile) {
    case 0: return launch_tile<tile_w(0), tile_h(0)>(gp, g.lds_bytes, temporal, nchunks, s);
    case 1: return launch_tile<tile_w(1), tile_h(1)>(gp, g.lds_bytes, temporal, nchunks, s);
    case 2: return launch_tile<tile_w(2), tile_h(2)>(gp, g.lds_bytes, temporal, nchunks, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fz
