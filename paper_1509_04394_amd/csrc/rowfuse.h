// Row-marching fused kernel for the Harris chain (gray or RGB input,
// Gaussian 5x5 -> Sobel -> products -> 5x5 sums -> Harris -> threshold ->
// 3x3 suppression [-> frame difference]).
//
// Same computation as the LDS tile engine (same per-pixel expressions, so the
// outputs are identical bit for bit), organised for gfx950 wavefronts:
//   * a wavefront owns a strip of 64*K columns (K adjacent columns per lane)
//     of a band of rows of one frame and marches down the rows; every window
//     stage keeps the few rows it still needs in registers (rings of 2r+1
//     rows; the 5x5 window sums keep sums of row pairs instead, and share
//     the pair sums of neighbouring columns across lanes), so nothing is
//     staged in LDS and no barrier is needed between rows;
//   * horizontal neighbours come from the adjacent lanes through DPP wave
//     shifts; a lane at the strip's edge receives its own edge value, which is
//     exactly the replicate border when the strip touches the frame edge (and a
//     don't-care halo value inside the frame, where the strips overlap by the
//     chain's horizontal halo);
//   * the row loop is unrolled by 15 (the least common multiple of the ring
//     sizes 3 and 5) so every ring slot is a fixed register;
//   * vertical replicate borders: when a stage produces the first row of the
//     frame it also writes it into the ring slots of the rows above, and after
//     the last row it copies it into the slots of the rows below, one slot per
//     iteration, once the consumer no longer needs the slot's old row;
//   * the suppression mask feeds the frame difference through the previous
//     frame's mask bits, packed in LDS; a work item covers a run of frames.
//     The difference at the first frame of a run needs the mask of the frame
//     before it, which the item of the previous run computes anyway: the two
//     items meet at their shared frame boundary (see row_exchange) instead of
//     the later one computing that frame again.  Without the exchange buffers
//     an item first recomputes the frame before its run (one frame of
//     temporal halo).
// The input rows are prefetched two iterations ahead.
#pragma once

#include <type_traits>

#include "engine.h"
#include "rowgeom.h"

namespace fz {

constexpr int ROW_UNROLL = 15;  // lcm of the ring sizes

// How one clip is split into work items.
struct RowGeom {
    int nstrips, nbands, nchunks, total;
    int strip_step;  // 64K - 2*ROW_HX
    int band_h;
    int tt;          // frames per work item
    // frame-boundary exchange (frame difference; null: recompute the frame
    // before each run instead): per boundary between runs c-1 and c of one
    // strip and band, two mask areas of 64 words a mask group (the earlier
    // run's last frame, the later run's first frame) and one arrival counter,
    // zeroed before the launch
    uint32_t* xmask;
    uint32_t* xcount;
};
struct RowParams {
    SegParams sp;
    RowGeom g;
};

// Value of the lane to the left (wave_shr:1) / right (wave_shl:1).  At a
// frame edge (EDGE) the edge lane keeps `edge`, its own edge column: the
// replicate border.  Inside the frame the edge lane is a halo lane whose value
// is never used, so it may read zero, which lets the compiler fold the shift
// into the instruction that consumes it.
template <bool EDGE>
__device__ __forceinline__ float dpp_from_left(float v, float edge)
{
    if constexpr (EDGE)
        return __int_as_float(
            __builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xf, 0xf, false));
    else
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xf, 0xf, true));
}
template <bool EDGE>
__device__ __forceinline__ float dpp_from_right(float v, float edge)
{
    if constexpr (EDGE)
        return __int_as_float(
            __builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
    else
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x130, 0xf, 0xf, true));
}

// e[0 .. K+2R) = this lane's columns x-R .. x+K-1+R of a row held K per lane.
// EL / ER: the strip's first / last column is the frame's.
template <int K, int R, bool EL, bool ER>
__device__ __forceinline__ void extend_row(const float (&v)[K], float (&e)[K + 2 * R])
{
    static_assert(R <= K, "neighbour lanes must hold the halo");
#pragma unroll
    for (int k = 0; k < K; ++k) e[R + k] = v[k];
#pragma unroll
    for (int i = 1; i <= R; ++i) {
        e[R - i] = dpp_from_left<EL>(v[K - i], v[0]);
        e[R + K - 1 + i] = dpp_from_right<ER>(v[i - 1], v[K - 1]);
    }
}

// Horizontal pass of the 5-wide window sum of a row held K per lane:
// s[k] = sum5(e[k], ..., e[k+4]) over the extended row e = extend_row<K, 2>(v),
// computed from pair sums p[j] = e[j] + e[j+1].  Window k needs p[k], p[k+2]
// and e[k+4]; each pair of adjacent columns is added once, by the lane that
// holds its right column, and a lane reads its neighbours' pairs through DPP
// shifts: p[0] is the left lane's p[K] and p[K+1] the right lane's p[1].  At
// a frame edge the shifted pair of the edge lane is the sum of its own edge
// column with itself, which is what the replicate border gives.  Same bits as
// sum5 on extend_row's output.
template <int K, bool EL, bool ER>
__device__ __forceinline__ void box5_row(const float (&v)[K], float (&s)[K])
{
    static_assert(K >= 2, "two or more columns per lane");
    float p[K + 2];
    p[1] = dpp_from_left<EL>(v[K - 1], v[0]) + v[0];  // straddles the left lane boundary
#pragma unroll
    for (int j = 2; j <= K; ++j) p[j] = v[j - 2] + v[j - 1];
    p[0] = dpp_from_left<EL>(p[K], p[1]);  // at the left frame edge p[1] = v[0] + v[0]
    p[K + 1] = dpp_from_right<ER>(p[1], ER ? v[K - 1] + v[K - 1] : 0.0f);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float e4 = k + 2 < K ? v[k + 2] : dpp_from_right<ER>(v[k + 2 - K], v[K - 1]);
        s[k] = (p[k] + p[k + 2]) + e4;
    }
}

// Raw buffer over `bytes` bytes at `base`: a store whose offset is at or past
// `bytes` is dropped by the hardware, which lets every lane issue its store
// with no divergent branch (columns outside the strip's output range get an
// out-of-range offset).  Word 3 selects 32-bit raw access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t out_rsrc(void* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, (int)bytes, 0x00020000);
}
constexpr int DROP = 0x7fffffff;  // an offset past any frame

template <int K>
__device__ __forceinline__ void copy_row(float (&d)[K], const float (&s)[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k) d[k] = s[k];
}

// NB consecutive input bytes kept as loaded: whole dwords, then a short,
// then a byte.  The short and the byte keep their 16- and 8-bit types so that
// their zero extension happens where they are used, not right after the
// load (an operation on a loaded register makes the wavefront wait for the
// load).
template <int NB>
struct RawRow {
    static constexpr int ND = NB / 4;
    uint32_t d[ND > 0 ? ND : 1];
    uint16_t h;  // bytes 4*ND, 4*ND+1 when NB % 4 >= 2
    uint8_t y;   // the last byte when NB is odd
};

template <int K, bool RGB>
struct RowState {
    static constexpr int NB = RGB ? 3 * K : K;  // input bytes per lane and row
    float h[5][K];     // Gaussian horizontal pass
    float g[3][K];     // Gaussian output
    float bp[3][K];    // window-sum horizontal pass of the previous row, 3 channels
    float q[3][3][K];  // pairs of consecutive horizontal-pass rows, q_r = b_r + b_(r+1)
    float rt[3][K];    // thresholded response
    float m[3][K];     // 3-wide horizontal maximum of rt
    RawRow<NB> raw[3];  // input rows, two loaded ahead
    uint32_t mask, prev;  // this mask group's suppression bits, and the previous frame's
};

struct RowCtx {
    const uint8_t* in_frame;  // frame t of the input
    uint8_t* out_frame;       // frame t of the output
    int W, Hf, x0, lane, y0, y1, t;
    int row_bytes;            // bytes per input row
    int lane_in, lane_out;    // byte offset of this lane's first column in an input / output row
    bool pts;                 // frame t's feature points are wanted
    bool store;               // its output is written now (not at a frame boundary exchange)
    uint32_t valid;           // bit k: column k of this lane is an output column of the strip
    int lo_in, hi_in, lo_g, hi_g, lo_s, hi_s, lo_b, hi_b;
    // iteration j computes a stage's row iff (unsigned)(j - j*) < n*: the rows
    // [lo, hi) of each stage mapped to iterations (row = y0 - 6 + j - lag)
    int jp, np_, ji, ni, jg, ng, js, ns, jq, nq, jb, nb, jn, nn;
    uint8_t* prev;            // LDS mask words of this wavefront, at this lane (DIFF)
    uint32_t diff;            // all ones; zero on the clip's first frame, whose difference is zero
    uint32_t tag;             // frame t's number in the item << 16 (feature points)
};

// NB consecutive bytes at byte offset voff + soff of buffer r into a RawRow:
// the fewest dword / short / byte loads; the bytes need not be aligned.  soff
// is wavefront-uniform (a scalar register), voff the lane's own offset, so
// the address needs no per-lane arithmetic.  byte_of<NB, I>(w) extracts byte
// I; keeping the bytes packed holds a row of 6 RGB bytes in 2 registers
// instead of 6.
template <int NB>
__device__ __forceinline__ void load_words(__amdgpu_buffer_rsrc_t r, int voff, int soff, RawRow<NB>& w)
{
    constexpr int D = NB / 4;
#pragma unroll
    for (int i = 0; i < D; ++i) w.d[i] = __builtin_amdgcn_raw_buffer_load_b32(r, voff + 4 * i, soff, 0);
    if constexpr (NB % 4 >= 2) w.h = __builtin_amdgcn_raw_buffer_load_b16(r, voff + 4 * D, soff, 0);
    if constexpr (NB % 2 == 1) w.y = __builtin_amdgcn_raw_buffer_load_b8(r, voff + NB - 1, soff, 0);
}
template <int NB, int I>
__device__ __forceinline__ uint32_t byte_of(const RawRow<NB>& w)
{
    constexpr int D = NB / 4;  // whole dwords
    if constexpr (I < 4 * D) return (w.d[I / 4] >> (8 * (I % 4))) & 0xffu;
    else if constexpr (NB % 4 >= 2 && I < 4 * D + 2) return ((uint32_t)w.h >> (8 * (I - 4 * D))) & 0xffu;
    else return (uint32_t)w.y;
}

// byte_of with the index as an argument (constant after unrolling).
template <int NB>
__device__ __forceinline__ uint32_t byte_at(const RawRow<NB>& w, int i)
{
    constexpr int D = NB / 4;
    if (i < 4 * D) return (w.d[i / 4] >> (8 * (i % 4))) & 0xffu;
    if (NB % 4 >= 2 && i < 4 * D + 2) return ((uint32_t)w.h >> (8 * (i - 4 * D))) & 0xffu;
    return (uint32_t)w.y;
}

// Gray value of each of the lane's K columns from its packed input bytes.
template <int K, bool RGB, int... k>
__device__ __forceinline__ void gray_row(const RawRow<RowState<K, RGB>::NB>& w, float (&gr)[K],
                                         std::integer_sequence<int, k...>)
{
    constexpr int NB = RowState<K, RGB>::NB;
    if constexpr (RGB)
        ((gr[k] = (float)rgb2gray(byte_of<NB, 3 * k>(w), byte_of<NB, 3 * k + 1>(w), byte_of<NB, 3 * k + 2>(w))), ...);
    else
        ((gr[k] = (float)byte_of<NB, k>(w)), ...);
}

// The K*C input bytes of this lane in input row `row`, packed.  The row is
// clamped into the frame (a wavefront-uniform scalar operation), so the load
// can be issued on every row step, in range, whether or not the row is used:
// an unconditional load lets the compiler count the loads still in flight
// and wait only for the one a step needs, instead of for all of them at the
// join after a conditional load.  Every strip lies inside the frame.
template <int K, bool RGB>
__device__ __forceinline__ void load_raw(const RowCtx& c, int row, RawRow<RowState<K, RGB>::NB>& raw)
{
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void*)c.in_frame, (short)0, c.row_bytes * c.Hf, 0x00020000);
    const int rc = row < 0 ? 0 : (row >= c.Hf ? c.Hf - 1 : row);
    load_words<RowState<K, RGB>::NB>(r, c.lane_in, rc * c.row_bytes, raw);
}

// 255 where bit `i` of w is set, else 0.
__device__ __forceinline__ uint8_t byte_mask(uint32_t w, int i) { return (uint8_t)((int32_t)(w << (31 - i)) >> 31); }

template <int K, bool RGB, bool DIFF, bool EL, bool ER, int U, class L>
__device__ __forceinline__ void row_step(RowState<K, RGB>& st, const RowCtx& c, const SegParams& p, L& list, int& ev,
                                         int j)
{
    constexpr int U3 = U % 3, U5 = U % 5;
    const int row_in = c.y0 - ROW_HX + j;

    // prefetch the input row two iterations ahead
    {
        const int rp = row_in + 2;
        load_raw<K, RGB>(c, rp, st.raw[(U + 2) % 3]);  // unused when rp is outside [lo_in, hi_in)
    }
    // Gaussian, horizontal pass, on the gray input row
    if ((unsigned)(j - c.ji) < (unsigned)c.ni) {
        float gr[K];
        gray_row<K, RGB>(st.raw[U3], gr, std::make_integer_sequence<int, K>{});
        float e[K + 4];
        extend_row<K, 2, EL, ER>(gr, e);
#pragma unroll
        for (int k = 0; k < K; ++k) st.h[U5][k] = gauss5_taps(p.gw, e[k], e[k + 1], e[k + 2], e[k + 3], e[k + 4]);
        if (row_in == 0) {
            copy_row<K>(st.h[(U + 4) % 5], st.h[U5]);
            copy_row<K>(st.h[(U + 3) % 5], st.h[U5]);
        }
    }
    // Gaussian, vertical pass: row row_in - 2
    const int rg = row_in - 2;
    if ((unsigned)(j - c.jg) < (unsigned)c.ng) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            st.g[U3][k] = gauss5_taps(p.gw, st.h[(U + 1) % 5][k], st.h[(U + 2) % 5][k], st.h[(U + 3) % 5][k],
                                      st.h[(U + 4) % 5][k], st.h[U5][k]);
        if (__builtin_expect(rg == 0, 0)) copy_row<K>(st.g[(U + 2) % 3], st.g[U3]);
    }
    // Sobel, products and the horizontal pass of the window sums: row row_in - 3
    const int rs = row_in - 3;
    float bn[3][K];  // horizontal pass of row rs
    if ((unsigned)(j - c.js) < (unsigned)c.ns) {
        float sv[K], ev[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float gm = st.g[(U + 1) % 3][k], g0 = st.g[(U + 2) % 3][k], gp = st.g[U3][k];
            sv[k] = sobel_sv(gm, g0, gp);
            ev[k] = sobel_e(gm, gp);
        }
        float esv[K + 2], eev[K + 2];
        extend_row<K, 1, EL, ER>(sv, esv);
        extend_row<K, 1, EL, ER>(ev, eev);
        float pr[3][K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float ix = sobel_ix(esv[k], esv[k + 2]);
            const float iy = sobel_iy(eev[k], eev[k + 1], eev[k + 2]);
            products(ix, iy, pr[0][k], pr[1][k], pr[2][k]);
        }
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) box5_row<K, EL, ER>(pr[ch], bn[ch]);
        if (rs == 0) {  // the row above the frame's first row is that row
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) copy_row<K>(st.bp[ch], bn[ch]);
        }
    } else {
        // below the frame's last row: the replicate border (elsewhere unused)
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) copy_row<K>(bn[ch], st.bp[ch]);
    }
    // Window sums (vertical), Harris, threshold, 3-wide maximum: row row_in - 5
    const int rb = row_in - 5;
    if ((unsigned)(j - c.jb) < (unsigned)c.nb) {
        // sum5 over rows rb-2 .. rb+2: (q_(rb-2) + q_rb) + b_(rb+2), the same
        // operations in the same order, with each row pair added once
        // (the pair of the two newest rows replaces q_(rb-2) right after its read)
        float s[3][K];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                s[ch][k] = (st.q[U3][ch][k] + st.q[(U + 2) % 3][ch][k]) + bn[ch][k];
                st.q[U3][ch][k] = st.bp[ch][k] + bn[ch][k];
            }
#pragma unroll
        for (int k = 0; k < K; ++k) st.rt[U3][k] = threshold(harris(s[0][k], s[1][k], s[2][k], p.k), p.thr);
        float e[K + 2];
        extend_row<K, 1, EL, ER>(st.rt[U3], e);
#pragma unroll
        for (int k = 0; k < K; ++k) st.m[U3][k] = max3(e[k], e[k + 1], e[k + 2]);
        if (rb == 0) {
            copy_row<K>(st.rt[(U + 2) % 3], st.rt[U3]);
            copy_row<K>(st.m[(U + 2) % 3], st.m[U3]);
        }
    }
    // Row pair q_(rs-1) = b_(rs-1) + b_rs on the iterations whose window sums
    // did not already form it (the first ones of the band); at the frame's
    // first row the two pairs above it are both twice row 0 (replicate border)
    if ((unsigned)(j - c.jq) < (unsigned)c.nq) {
#pragma unroll
        for (int ch = 0; ch < 3; ++ch)
#pragma unroll
            for (int k = 0; k < K; ++k) st.q[U3][ch][k] = st.bp[ch][k] + bn[ch][k];
        if (rs == 0) {
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) copy_row<K>(st.q[(U + 2) % 3][ch], st.q[U3][ch]);
        }
    }
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) copy_row<K>(st.bp[ch], bn[ch]);
    // Suppression, feature points, output: row row_in - 6
    const int rn = row_in - 6;
    if ((unsigned)(j - c.jn) < (unsigned)c.nn) {
        uint32_t bits = 0;
        float centre[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float wmax = max3(st.m[(U + 1) % 3][k], st.m[(U + 2) % 3][k], st.m[U3][k]);
            centre[k] = st.rt[(U + 2) % 3][k];
            bits |= (nms_keep(centre[k], wmax) != 0u ? 1u : 0u) << k;
        }
        const uint32_t pts = bits & c.valid;
        const unsigned long long pm = __ballot(pts != 0u);
        if (c.pts && pm != 0ull) list_put<K>(list, ev, pm, pts, (uint32_t)rn, (uint32_t)c.lane | c.tag, centre);
        uint32_t out = bits;  // the row's K bits from bit SH on
        constexpr int P = DIFF ? (U + 3) % ROW_UNROLL % row_mask_rows(K) : 0, SH = K * P;
        if constexpr (DIFF) {
            // row U of the unrolled loop is row P of its mask group
            static_assert(ROW_UNROLL % row_mask_rows(K) == 0 && 2 * ROW_HX == 12, "row places are constants");
            const int at = (rn - c.y0 - P) * row_mask_pitch(K);
            if (P == 0) {
                st.mask = bits;
                st.prev = *(uint32_t*)(c.prev + at);  // not used on the first frame marched
            } else {
                st.mask |= bits << SH;
            }
            if (P == row_mask_rows(K) - 1) *(uint32_t*)(c.prev + at) = st.mask;
            out = (st.mask ^ st.prev) & c.diff;
        }
        if (c.store) {
            const __amdgpu_buffer_rsrc_t r = out_rsrc(c.out_frame, (uint32_t)(c.W * c.Hf));
            const int soff = rn * c.W;  // uniform row offset
#pragma unroll
            for (int k = 0; k < K; ++k)
                __builtin_amdgcn_raw_buffer_store_b8(byte_mask(out, SH + k), r,
                                                     (c.valid >> k & 1u) ? c.lane_out + k : DROP, soff, 0);
        }
    }
    // bottom replicate of the Gaussian and response rings: after the last
    // frame row, copy it into the next slot, once per iteration, for as many
    // rows as the consumer reads (rare: branches, not selects on every row)
    if (__builtin_expect(row_in >= c.Hf - 1 && row_in <= c.Hf, 0)) copy_row<K>(st.h[(U + 1) % 5], st.h[U5]);
    if (__builtin_expect(rg == c.Hf - 1, 0)) copy_row<K>(st.g[(U + 1) % 3], st.g[U3]);
    if (rb == c.Hf - 1) {
        copy_row<K>(st.rt[(U + 1) % 3], st.rt[U3]);
        copy_row<K>(st.m[(U + 1) % 3], st.m[U3]);
    }
}

template <int K, bool RGB, bool DIFF, bool EL, bool ER, class L, int... U>
__device__ __forceinline__ void row_block(RowState<K, RGB>& st, const RowCtx& c, const SegParams& p, L& list, int& ev,
                                          int jb, int n, std::integer_sequence<int, U...>)
{
    ((jb + U < n ? row_step<K, RGB, DIFF, EL, ER, U>(st, c, p, list, ev, jb + U) : void()), ...);
}

// One side of a frame boundary between two runs of frames of the same strip
// and band: the mask of the frame next to the boundary on this side (the words
// in LDS) is published; the side that arrives second reads the other side's
// words and writes the frame difference of the later run's first frame
// (out_frame): the exclusive or of the two masks, the same bits the later item
// would have formed from a recomputed frame.  Neither side waits for the other.
//
// Every access to the exchange words and the counter is a device-scope
// atomic read-modify-write, which the device performs coherently across its
// XCDs; the words are published with exchanges whose results are waited for
// before the arrival is counted, and read (fetch-or 0) only after the count
// has come back.  No fence is used: an agent-scope release or acquire fence
// writes back or invalidates the XCD's whole L2, which cost the kernel a
// quarter of its speed (the strips of neighbouring items share input rows
// in L2).
//
// Words of 15 rows a lane, as the row loop packs them.  With a byte a lane and
// row in LDS and a ballot word a column and row in the exchange, forming and
// taking the words apart cost about 0.45 of a frame an item: 800x600x1000 RGB
// at 86 rows x 2 frames 1075 us (now 1016), gray 959 us (now 822; 764 without
// the frame difference), 192x432x600 gray at 30 x 2 171 us (now 156).
template <int K>
__device__ __forceinline__ void row_exchange(const RowCtx& c, uint32_t* mine, uint32_t* other, uint32_t* cnt,
                                             uint8_t* out_frame)
{
    constexpr int G = row_mask_rows(K), STEP = G * row_mask_pitch(K);
    constexpr int AHEAD = 6;  // words in flight
    const int nrow = c.y1 - c.y0, ng = (nrow + G - 1) / G;
    // the lane's number as a value of its own: addresses formed from it here
    // would otherwise be kept in registers all through the row loop
    int lane = c.lane;
    asm volatile("" : "+v"(lane));
    uint32_t sink = 0;
#pragma unroll 1
    for (int g = 0; g < ng; ++g)
        sink |= __hip_atomic_exchange(mine + g * 64 + lane, *(uint32_t*)(c.prev + g * STEP), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    // the exchanges have returned (so they are performed) before the arrival
    // is counted: the empty asm needs their results, and orders the memory
    // operations around it
    asm volatile("" ::"v"(sink) : "memory");
    uint32_t old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = __builtin_amdgcn_readfirstlane(old);
    if (old == 0u) return;
    const __amdgpu_buffer_rsrc_t rs = out_rsrc(out_frame, (uint32_t)(c.W * c.Hf));
#pragma unroll 1
    for (int g0 = 0; g0 < ng; g0 += AHEAD) {
        uint32_t w[AHEAD];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)  // past the last group: its words again
            w[i] = __hip_atomic_fetch_or(other + min(g0 + i, ng - 1) * 64 + lane, 0u, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int g = g0 + i;
            if (g >= ng) break;
            uint32_t x = w[i] ^ *(uint32_t*)(c.prev + g * STEP);
            const int nr = min(G, nrow - g * G);
            int soff = (c.y0 + g * G) * c.W;
#pragma unroll 1
            for (int r = 0; r < nr; ++r, soff += c.W, x >>= K) {
#pragma unroll
                for (int k = 0; k < K; ++k)
                    __builtin_amdgcn_raw_buffer_store_b8(byte_mask(x, k), rs,
                                                         (c.valid >> k & 1u) ? c.lane_out + k : DROP, soff, 0);
            }
        }
    }
}

// The geometry at byte `at` of the kernel arguments, as an address the compiler
// does not see through.
typedef const __attribute__((address_space(4))) RowGeom RowGeomK;
__device__ __forceinline__ RowGeomK* kernel_geom(int at)
{
    auto k = (RowGeomK*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + at);
    asm volatile("" : "+s"(k));
    return k;
}

// Exchange areas of the boundary before run `chunk` (chunk >= 1).
struct RowBoundary {
    uint32_t* last;   // the earlier run's last frame
    uint32_t* first;  // the later run's first frame
    uint32_t* cnt;
};
template <int K>
__device__ __forceinline__ RowBoundary row_boundary(RowGeomK& rp, int strip, int band, int chunk)
{
    const size_t b = ((size_t)(chunk - 1) * rp.nbands + band) * rp.nstrips + strip;
    const size_t words = (size_t)row_mask_groups(K, rp.band_h) * 64;
    return RowBoundary{rp.xmask + 2 * b * words, rp.xmask + (2 * b + 1) * words, rp.xcount + b};
}

// All frames of one work item.
template <int K, bool RGB, bool DIFF, bool EL, bool ER, class L>
__device__ __forceinline__ void row_frames(RowCtx& c, const SegParams& p, bool exchange, int geom_at, L& list, int& held,
                                           int strip, int band, int ts, int t0, int t1)
{
    constexpr int C = RGB ? 3 : 1;
    const size_t plane = (size_t)p.W * p.H;
    const int n = c.y1 - c.y0 + 2 * ROW_HX;
    const bool xch = DIFF && exchange;
    const bool want = p.count != nullptr;
    for (int t = ts; t < t1; ++t) {
        c.t = t;
        c.pts = t >= t0 && want;
        c.tag = (uint32_t)(t - t0) << 16;
        c.diff = t == 0 ? 0u : ~0u;
        c.in_frame = (const uint8_t*)p.in + (size_t)t * plane * C;
        c.out_frame = (uint8_t*)p.out + (size_t)t * plane;
        if (t > t0) list_room<K>(list, held, t - t0);
        march_points<K>(list, held, [&](int& ev, bool again) {
            c.store = t >= t0 && !(xch && t == t0 && t0 > 0) && !again;
            RowState<K, RGB> st;
            // first two input rows
            const int r0 = c.y0 - ROW_HX;
            load_raw<K, RGB>(c, r0, st.raw[0]);
            load_raw<K, RGB>(c, r0 + 1, st.raw[1]);
#pragma unroll 1
            for (int jb = 0; jb < n; jb += ROW_UNROLL)
                row_block<K, RGB, DIFF, EL, ER>(st, c, p, list, ev, jb, n,
                                                std::make_integer_sequence<int, ROW_UNROLL>{});
            if constexpr (DIFF) {  // the last mask group, where the band ends inside one
                const int part = (c.y1 - c.y0) % row_mask_rows(K);
                if (part != 0) *(uint32_t*)(c.prev + (c.y1 - c.y0 - part) * row_mask_pitch(K)) = st.mask;
            }
        });
        if constexpr (DIFF) {
            // (the launch's parameters are read again: kept through the row loop
            // they would spill other scalars into vector registers)
            if (xch && t == t0 && t0 > 0) {  // the boundary before the run: this side is its first frame
                RowGeomK& k = *kernel_geom(geom_at);
                const RowBoundary x = row_boundary<K>(k, strip, band, t / k.tt);
                row_exchange<K>(c, x.first, x.last, x.cnt, c.out_frame);
            }
            if (xch && t == t1 - 1 && t1 < p.T) {  // the boundary after the run: this side is its last frame
                RowGeomK& k = *kernel_geom(geom_at);
                const RowBoundary x = row_boundary<K>(k, strip, band, (t + 1) / k.tt);
                row_exchange<K>(c, x.last, x.first, x.cnt, c.out_frame + (size_t)c.W * c.Hf);
            }
        }
    }
}

// Geometry of one work item: strip, band and frame run of one clip.
struct RowItem {
    int strip, band, chunk;
    int nstrips, band_h, tt, strip_step;
};

// One work item of one wavefront (all of it wavefront-uniform).  geom_at: the
// byte of its RowGeom in the kernel arguments; exchange: whether that has
// exchange buffers.  Returns the entries left in its point list.
template <int K, bool RGB, bool DIFF, class L>
__device__ __forceinline__ int row_item(const SegParams& p, const RowItem& it, bool exchange, int geom_at,
                                        uint8_t* prev_lds, L& list)
{
    RowCtx c;
    c.W = p.W;
    c.Hf = p.H;
    c.lane = threadIdx.x & 63;
    const int S = it.strip_step;
    c.x0 = min(it.strip * S, p.W - 64 * K);
    constexpr int CIN = RGB ? 3 : 1;
    c.row_bytes = p.W * CIN;
    c.lane_in = (c.x0 + K * c.lane) * CIN;
    c.lane_out = c.x0 + K * c.lane;
    const int vx0 = it.strip == 0 ? 0 : (it.strip - 1) * S + 64 * K - ROW_HX;
    const int vx1 = it.strip == it.nstrips - 1 ? p.W : it.strip * S + 64 * K - ROW_HX;
    c.valid = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int x = c.x0 + K * c.lane + k;
        c.valid |= (x >= vx0 && x < vx1 ? 1u : 0u) << k;
    }
    c.y0 = it.band * it.band_h;
    c.y1 = min(c.y0 + it.band_h, p.H);
    c.lo_in = max(0, c.y0 - 6);
    c.hi_in = min(p.H, c.y1 + 6);
    c.lo_g = max(0, c.y0 - 4);
    c.hi_g = min(p.H, c.y1 + 4);
    c.lo_s = max(0, c.y0 - 3);
    c.hi_s = min(p.H, c.y1 + 3);
    c.lo_b = max(0, c.y0 - 1);
    c.hi_b = min(p.H, c.y1 + 1);
    // row r of a stage with lag L (rows behind the input row) is computed at
    // iteration j = r - y0 + 6 + L
    const int base = ROW_HX - c.y0;
    c.jp = c.lo_in + base - 2;  // prefetch of row j + 2
    c.np_ = c.hi_in - c.lo_in;
    c.ji = c.lo_in + base;
    c.ni = c.hi_in - c.lo_in;
    c.jg = c.lo_g + base + 2;
    c.ng = c.hi_g - c.lo_g;
    c.js = c.lo_s + base + 3;
    c.ns = c.hi_s - c.lo_s;
    c.jb = c.lo_b + base + 5;
    c.nb = c.hi_b - c.lo_b;
    // row pairs q_(s-1): the window sums of rows [lo_b, hi_b) read q_(lo_b-2) ..
    // q_(hi_b-1), formed on the iterations s = max(lo_b - 1, lo_s) .. hi_b; from
    // s = lo_b + 2 on, the window-sum step forms them, so the pair step runs on
    // the iterations before it
    const int lo_q = max(c.lo_b - 1, c.lo_s);
    c.jq = lo_q + base + 3;
    c.nq = c.lo_b + 2 - lo_q;
    c.jn = c.y0 + base + 6;
    c.nn = c.y1 - c.y0;
    c.prev = prev_lds + 4 * c.lane;

    const int t0 = it.chunk * it.tt;
    const int t1 = min(t0 + it.tt, p.T);
    const int ts = (DIFF && t0 > 0 && !exchange) ? t0 - 1 : t0;
    list_begin<K>(list, p, c.x0, t0);
    int held = 0;
    const bool el = it.strip == 0, er = it.strip == it.nstrips - 1;
    if constexpr (std::is_same_v<L, PointDirect>)
        row_frames<K, RGB, DIFF, true, true>(c, p, exchange, geom_at, list, held, it.strip, it.band, ts, t0, t1);
    else if (el && er)
        row_frames<K, RGB, DIFF, true, true>(c, p, exchange, geom_at, list, held, it.strip, it.band, ts, t0, t1);
    else if (el)
        row_frames<K, RGB, DIFF, true, false>(c, p, exchange, geom_at, list, held, it.strip, it.band, ts, t0, t1);
    else if (er)
        row_frames<K, RGB, DIFF, false, true>(c, p, exchange, geom_at, list, held, it.strip, it.band, ts, t0, t1);
    else
        row_frames<K, RGB, DIFF, false, false>(c, p, exchange, geom_at, list, held, it.strip, it.band, ts, t0, t1);
    return held;
}

// Decompose a clip-local item index.  Strips vary fastest, then bands, then
// frame runs: the wavefronts in flight cover whole frames, neighbouring
// wavefronts reading neighbouring segments of the same rows.  (With strips
// varying slowest, the wavefronts in flight covered one 128-column strip of
// hundreds of frames, and the memory-bound kernels ran at a third of the
// bandwidth.)
__device__ __forceinline__ RowItem row_decompose(int item, int nstrips, int nbands, int nchunks, int band_h, int tt,
                                                 int strip_step)
{
    RowItem it;
    it.strip = item % nstrips;
    const int rest = item / nstrips;
    it.band = rest % nbands;
    it.chunk = rest / nbands;
    it.nstrips = nstrips;
    it.band_h = band_h;
    it.tt = tt;
    it.strip_step = strip_step;
    return it;
}

template <int K, bool RGB, bool DIFF>
__global__ __launch_bounds__(ROW_WAVES * 64, K == 2 ? (RGB ? 5 : 6) : 4) void k_rowfuse(RowParams rp)
{
    extern __shared__ uint8_t row_lds[];
    __shared__ PointLists<K, ROW_WAVES> lists;
    static_assert(sizeof(lists) == row_list_bytes(K), "the planner counts these bytes");
    lists_begin(lists);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wavefront-uniform
    const int item = blockIdx.x * ROW_WAVES + wave;
    if (item >= rp.g.total) return;  // whole wavefront leaves; no barrier is used from here on
    const RowItem it =
        row_decompose(item, rp.g.nstrips, rp.g.nbands, rp.g.nchunks, rp.g.band_h, rp.g.tt, rp.g.strip_step);
    const int held = row_item<K, RGB, DIFF>(rp.sp, it, rp.g.xcount != nullptr, offsetof(RowParams, g),
                                            row_lds + wave * row_mask_bytes(K, rp.g.band_h), lists.wave[wave]);
    if (rp.sp.count != nullptr)
        lists_end(lists, wave, held, min(ROW_WAVES, rp.g.total - (int)blockIdx.x * ROW_WAVES));
}

// The same for plans whose LDS budget does not hold the lists.  (One form of the
// row loop for every strip: an interior strip's border values are not used.)
template <int K, bool RGB, bool DIFF>
__global__ __launch_bounds__(ROW_WAVES * 64) void k_rowfuse_direct(RowParams rp)
{
    extern __shared__ uint8_t row_lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int item = blockIdx.x * ROW_WAVES + wave;
    if (item >= rp.g.total) return;
    const RowItem it =
        row_decompose(item, rp.g.nstrips, rp.g.nbands, rp.g.nchunks, rp.g.band_h, rp.g.tt, rp.g.strip_step);
    PointDirect list;
    (void)row_item<K, RGB, DIFF>(rp.sp, it, rp.g.xcount != nullptr, offsetof(RowParams, g),
                                 row_lds + wave * row_mask_bytes(K, rp.g.band_h), list);
}

// ---------------------------------------------------------------- batches
// Many clips of different sizes in one launch: the clips' workgroups are
// numbered clip after clip, and a workgroup runs the items of one clip exactly
// as the single-clip kernel does (frame-boundary exchange and point lists
// included).  Clip descriptors travel by value in the kernel arguments.
//
// (Wavefronts that took 16-frame items of 64 rows from a queue counter, each
// recomputing the frame before its run, ran 16 gray clips of 1.2 Gpixel in 2.81
// ms; now 2.09 ms, the single-clip kernel's rate.)
constexpr int FZ_BATCH_MAX = 32;
constexpr int BATCH_TT = 4;  // frames per item: a run's exchange words are 8% of its input

struct BatchClip {
    const void* in;
    void* out;
    fz_point* points;
    uint32_t* count;
    int W, H, T;
    uint32_t cap;
    int wg_begin;  // first workgroup
    RowGeom g;
};

struct BatchParams {
    Gauss5W gw;
    float k, thr;
    int n_clips, max_band;  // tallest band of the clips
    uint32_t* counters;     // the clips' arrival counters, one after another, zero at launch
    int n_counters;
    BatchClip clip[FZ_BATCH_MAX];
};
static_assert(sizeof(BatchParams) <= 4096, "kernel arguments must stay within 4 KB");

template <int K, bool RGB, bool DIFF>
__global__ __launch_bounds__(ROW_WAVES * 64, RGB ? 5 : 6) void k_rowfuse_batch(BatchParams)
{
    extern __shared__ uint8_t row_lds[];
    __shared__ PointLists<K, ROW_WAVES> lists;
    lists_begin(lists);
    typedef const __attribute__((address_space(4))) BatchParams BatchParamsK;
    BatchParamsK& bp = *(BatchParamsK*)__builtin_amdgcn_kernarg_segment_ptr();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wg = blockIdx.x;
    int ci = 0;
    while (ci + 1 < bp.n_clips && wg >= bp.clip[ci + 1].wg_begin) ++ci;
    const auto& bc = bp.clip[ci];
    const int first = (wg - bc.wg_begin) * ROW_WAVES, item = first + wave;
    if (item >= bc.g.total) return;
    SegParams sp;
    sp.in = bc.in;
    sp.out = bc.out;
    sp.W = bc.W;
    sp.H = bc.H;
    sp.T = bc.T;
    sp.tpb = bc.g.tt;
    sp.gw.w0 = bp.gw.w0;
    sp.gw.w1 = bp.gw.w1;
    sp.gw.w2 = bp.gw.w2;
    sp.k = bp.k;
    sp.thr = bp.thr;
    sp.points = bc.points;
    sp.count = bc.count;
    sp.cap = bc.cap;
    const RowItem it = row_decompose(item, bc.g.nstrips, bc.g.nbands, bc.g.nchunks, bc.g.band_h, bc.g.tt, bc.g.strip_step);
    const int held = row_item<K, RGB, DIFF>(
        sp, it, bc.g.xcount != nullptr, (int)(offsetof(BatchParams, clip) + ci * sizeof(BatchClip) + offsetof(BatchClip, g)),
        row_lds + wave * row_mask_bytes(K, bp.max_band), lists.wave[wave]);
    if (sp.count != nullptr) lists_end(lists, wave, held, min(ROW_WAVES, bc.g.total - first));
}

// Tall bands: the mask rows and the point lists pass the 64 KB a workgroup has
// by default (the CU has 160 KB).
inline hipError_t allow_row_lds(const void* kernel, size_t mask_rows)
{
    if (mask_rows + sizeof(PointLists<3, ROW_WAVES>) <= 65536) return hipSuccess;
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)mask_rows);
}

hipError_t launch_rowfuse_batch(const BatchParams& bp, bool rgb, bool diff, int blocks, hipStream_t s);

hipError_t launch_rowfuse(const RowParams& rp, int K, bool rgb, bool diff, hipStream_t s);
hipError_t launch_rowfuse_direct(const RowParams& rp, int K, bool rgb, bool diff, hipStream_t s);

// Zero n words (the frame-boundary arrival counters) and the point count (null:
// none); a kernel, not a memset, so that it is an ordinary kernel node when a run
// is captured into a graph.
hipError_t zero_words(uint32_t* p, int n, uint32_t* count, hipStream_t s);

template <bool LISTS, int K, bool RGB, bool DIFF>
hipError_t launch_rowfuse_t(const RowParams& rp, hipStream_t s)
{
    const int blocks = (rp.g.total + ROW_WAVES - 1) / ROW_WAVES;
    const size_t lds = DIFF ? (size_t)ROW_WAVES * row_mask_bytes(K, rp.g.band_h) : 0;
    const int nb = DIFF && rp.g.xcount != nullptr ? row_boundaries(rp.g.nstrips, rp.g.nbands, rp.g.nchunks) : 0;
    hipError_t e = nb > 0 || rp.sp.count != nullptr ? zero_words(rp.g.xcount, nb, rp.sp.count, s) : hipSuccess;
    if (e != hipSuccess) return e;
    auto go = [&](auto kern) {
        if ((e = allow_row_lds((const void*)kern, lds)) != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(ROW_WAVES * 64), lds, s, rp);
        return hipGetLastError();
    };
    if constexpr (LISTS)
        return go(k_rowfuse<K, RGB, DIFF>);
    else
        return go(k_rowfuse_direct<K, RGB, DIFF>);
}
template <bool LISTS>
hipError_t pick_rowfuse(const RowParams& rp, int K, bool rgb, bool diff, hipStream_t s)
{
    hipError_t (*fn)(const RowParams&, hipStream_t) = nullptr;
    if (K == 2 && rgb) fn = diff ? launch_rowfuse_t<LISTS, 2, true, true> : launch_rowfuse_t<LISTS, 2, true, false>;
    if (K == 2 && !rgb) fn = diff ? launch_rowfuse_t<LISTS, 2, false, true> : launch_rowfuse_t<LISTS, 2, false, false>;
    if (K == 3 && rgb) fn = diff ? launch_rowfuse_t<LISTS, 3, true, true> : launch_rowfuse_t<LISTS, 3, true, false>;
    if (K == 3 && !rgb) fn = diff ? launch_rowfuse_t<LISTS, 3, false, true> : launch_rowfuse_t<LISTS, 3, false, false>;
    return fn ? fn(rp, s) : hipErrorInvalidValue;
}

}  // namespace fz
