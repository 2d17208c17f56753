// Geometry of the row-marching kernel, shared by the planner and the launcher.
#pragma once

#include <algorithm>
#include <cmath>

#include "fz_ops.h"

namespace fz {

constexpr int ROW_HX = 6;     // horizontal and vertical halo of the chain: 2 + 1 + 2 + 1
constexpr int ROW_WAVES = 4;  // independent wavefronts per workgroup
// Wavefronts per SIMD of the Harris row kernel (512 registers per lane, allocated in
// blocks of 8; the kernel's launch bounds ask for these): two columns per lane
// take 86 registers with RGB input (5 waves) and 80 with gray input (6 waves; two
// or three more go to 8-12 bytes of scratch a lane with the frame difference: at 5
// waves without them 192x432x600 takes 143 us, at 6 with them 136, the 16-clip
// batch 2.23 and 2.10 ms), three columns <= 123 (4 waves).
inline int row_waves(int K, bool rgb) { return K == 3 ? 4 : (rgb ? 5 : 6); }
// Wavefronts the 256 CUs (4 SIMDs each) hold at once; 4 per SIMD is assumed
// for the generic row kernel.
inline int row_slots(int K, bool rgb) { return 256 * 4 * row_waves(K, rgb); }
constexpr int ROW_SLOTS_GENERIC = 256 * 4 * 4;

// Groups the row kernel implements: gray conversion or Gaussian first, suppression
// or frame difference last, of the Harris chain.
constexpr bool row_group(int ch, int A, int B) { return ch == CHAIN_HARRIS && (A == 0 || A == 1) && (B == 7 || B == 8); }

// Strips of 64*K columns that overlap by 2*halo cover a frame of width W.
inline int row_strips(int W, int K, int halo = ROW_HX)
{
    const int span = 64 * K, S = span - 2 * halo;
    if (W < span) return 0;
    return 1 + (W - span + S - 1) / S;
}

// Groups the generic row kernel implements: any group with a window stage
// (one column per lane pair, K = 2).
inline bool rowgen_group(int ch, int A, int B) { return group_has_window(ch, A, B); }

// Columns per lane (2 or 3): the choice that computes the fewest columns per
// wavefront the SIMDs can hold; 0 if the frame is narrower than 128 columns.
inline int row_strips_best(int W, bool rgb)
{
    const int n2 = row_strips(W, 2), n3 = row_strips(W, 3);
    if (n2 == 0) return 0;
    if (n3 > 0 && n3 * 192 * row_waves(2, rgb) < n2 * 128 * row_waves(3, rgb)) return 3;
    return 2;
}

// Suppression mask of a band on the frame-difference kernels: a lane packs its
// K bits of ROW_MASK_ROWS consecutive rows into one word (the row loop is
// unrolled by 15, so a row's place in its word is a constant), and the words of
// ROW_MASK_ROWS rows are ROW_MASK_ROWS * row_mask_pitch bytes apart in LDS (a
// multiple of the row number, without a division).
constexpr int row_mask_rows(int K) { return K == 2 ? 15 : 5; }
constexpr int row_mask_pitch(int K) { return K == 2 ? 20 : 52; }  // >= 256 / row_mask_rows, bytes a row
constexpr int row_mask_groups(int K, int band_h) { return (band_h + row_mask_rows(K) - 1) / row_mask_rows(K); }
constexpr int row_mask_bytes(int K, int band_h)
{
    return row_mask_groups(K, band_h) * row_mask_rows(K) * row_mask_pitch(K);
}
// The on-chip memory a plan states for a frame-difference row group: a byte a
// lane and row.  What the kernels hold is row_held_bytes; a plan's budget has to
// cover both.
inline int row_lds_bytes(int band_h) { return ROW_WAVES * band_h * 64; }
// The feature-point lists of a workgroup (PointLists, groups with the suppression stage).
constexpr int row_list_bytes(int K) { return ROW_WAVES * (256 * (2 + K) + 32) + 8; }
// LDS of a row group's workgroup: the previous frame's mask of a frame-difference
// group (bytes in the generic kernel, packed words in the Harris kernel), and the
// point lists where the points are collected.
constexpr int row_held_bytes(bool generic, int K, int band_h, bool diff, bool lists)
{
    return (diff ? ROW_WAVES * (generic ? 64 * band_h : row_mask_bytes(K, band_h)) : 0) + (lists ? row_list_bytes(K) : 0);
}

// A frame-difference group's bands have at most this many rows: one byte of
// previous-frame mask bits per lane and band row in LDS (64 * band_h per
// wavefront) is then at most 64 KB for a workgroup of ROW_WAVES wavefronts.
constexpr int ROW_DIFF_MAX_BAND = 256;
// Wavefronts at once of the Harris row kernel: `slots` as its registers allow, or
// those of the workgroups the LDS holds (three columns a lane, bands over 170
// rows: 365x800x10000 RGB at 200 rows 6.47 ms, at 160 5.58).
inline int row_resident(int slots, int K, int band_h, bool diff)
{
    return std::min(slots, 256 * ROW_WAVES * (163840 / row_held_bytes(false, K, band_h, diff, true)));
}
// The tallest band within `budget` bytes of LDS, stated and held (0: none).
inline int row_tallest_band(bool generic, int K, bool diff, bool lists, int budget)
{
    if (!diff) return row_held_bytes(generic, K, 0, false, lists) <= budget ? 1 << 30 : 0;
    int b = ROW_DIFF_MAX_BAND;
    while (b > 0 && std::max(row_lds_bytes(b), row_held_bytes(generic, K, b, true, lists)) > budget) --b;
    return b;
}

// Frame boundaries between consecutive runs of one strip and band, and the
// device bytes of their exchange (two areas of a word a lane and mask group and
// one counter each, 256-byte aligned), for a frame-difference row group.
FZ_HD inline int row_boundaries(int nstrips, int nbands, int nchunks)
{
    return nchunks > 1 ? nstrips * nbands * (nchunks - 1) : 0;
}
inline size_t row_exchange_bytes(int nstrips, int nbands, int nchunks, int band_h, int K)
{
    const size_t nb = (size_t)row_boundaries(nstrips, nbands, nchunks);
    return nb == 0 ? 0 : 2 * nb * row_mask_groups(K, band_h) * 256 + ((nb * 4 + 255) & ~(size_t)255);
}

// Rows per band and frames per work item, from a model of the launch's time.
//
// Harris row kernel: an item of b rows x t frames takes
//   w = (b + 8.9) (t + 0.15) + 9.7
// row times (12 halo rows of which the first run only the first stages; the
// frame-boundary exchange, 0.15 of a frame where there is one; the item's
// start and end), and a launch of r = items / (wavefronts at once) rounds
//   w (r + 0.083 (ceil(r) - r) + 0.9):
// the work itself, part of the last round's idle share, and the first round's
// latency, with few wavefronts a SIMD to hide it.  The five constants fit a
// measured sweep (bands 4-160 x runs 1-8, 28 clips of 150x70x500 to
// 800x600x1000, RGB and gray, with and without the frame difference): the
// shape it picks is 0.9% slower than the best of the sweep on average, 4.5% at
// worst.  Its predecessor, (b + 12) (t + 0.45) (1 + 1/r) with bands from 16
// rows on, lost 11.7% on average and 27% on the smallest clips (320x240x4 RGB:
// 16 rows 30.0 us, 4 rows 21.9; 800x600x200 RGB: 30 x 2 269 us, 67 x 1 246).
//
// Generic row kernel: without a frame difference, the height nearest 18 rows
// that divides the frame evenly; under two rounds, of the heights nearest 14, 15
// and 16 the one with the fewest rows one after another on the compute unit that
// gets the most workgroups.  (A sweep over eight groups x eight clips is flat and
// memory-bound around 18: on clips over 2 Mpixel it is 4% from each case's best on
// average, the model that follows 10%.  On fourteen smaller clips x seventeen
// groups, 14 alone was up to 20% slower than 16 where it gave a compute unit a
// third workgroup: 333x251x40 gray conversion to products 21.0 us, 17.0 at 15
// rows; at 192x432x64 14 rows are 7% faster.  The rule is 14% from the sweep's
// best there, 14 alone 16%, the model that follows 19%.)  With one, the total work,
// items x (b + 12) x (t + 0.45), times (1 + 1/r), bands from 16 rows on.
// Explicit requests (> 0)
// are kept as given, except that a frame run longer than the video is the
// whole video and a band taller than the frame the whole frame; a request the
// kernel cannot run (a band over ROW_DIFF_MAX_BAND rows on a frame-difference
// group) gives band_h = 0 and is refused by the caller, never replaced.  Bands
// of the planner's choice have at most max_band rows (LDS); where none can, band_h
// is 0 too.
struct RowShape {
    int band_h, tt;
};
// The model's time of `items` items of bh rows that march `frames` frames.
inline double row_time(int bh, double frames, double items, int slots)
{
    const double r = items / (double)slots, w = (bh + 8.9) * frames + 9.7;
    return w * (r + 0.083 * (std::ceil(r) - r) + 0.9);
}
inline RowShape row_shape(int H, int T, int nstrips, bool diff, int req_h, int req_tt, int slots, bool generic, int max_band,
                          int K)
{
    if (req_h > 0 && diff && std::min(req_h, H) > ROW_DIFF_MAX_BAND) return RowShape{0, 0};
    if (req_h <= 0 && max_band < 1) return RowShape{0, 0};
    if (generic && !diff && req_h <= 0) {
        auto even = [&](int rows) {
            const int nb = std::max(1, (H + rows / 2) / rows);
            return (H + nb - 1) / nb;
        };
        int bh = even(18);
        auto items = [&](int rows) { return (long long)nstrips * ((H + rows - 1) / rows) * T; };
        if (items(bh) < 2LL * slots) {
            // rows one after another on the compute unit with the most workgroups
            auto chain = [&](int rows) { return rows * ((items(rows) + 256 * ROW_WAVES - 1) / (256 * ROW_WAVES)); };
            bh = even(14);
            for (int rows : {15, 16})
                if (chain(even(rows)) < chain(bh)) bh = even(rows);
        }
        return RowShape{bh, req_tt > 0 ? std::min(req_tt, T) : 1};
    }
    RowShape best{0, 0};
    double best_cost = -1.0;
    const int tts[] = {1, 2, 3, 4, 8, 16, 32, 64}, least = generic ? 16 : 4;
    for (int tt : tts) {
        int t = tt;
        if (req_tt > 0) {
            if (tt != 1) break;
            t = std::min(req_tt, T);
        } else if ((!diff && t != 1) || (t > T && t != 1)) {
            continue;
        }
        for (int nb = 1, last = 0; nb <= H; ++nb) {
            const int bh = req_h > 0 ? std::min(req_h, H) : (H + nb - 1) / nb;
            if (bh == last || (req_h <= 0 && bh > max_band)) continue;
            last = bh;
            if (bh < least && req_h <= 0 && nb > 1) break;
            const long long items = (long long)nstrips * ((H + bh - 1) / bh) * ((T + t - 1) / t);
            const double xch = diff && t < T ? 1.0 : 0.0;
            double cost;
            if (generic) {
                // the mask rows in LDS (a byte a lane and row) can hold fewer wavefronts than the registers
                long long fit = slots;
                if (diff) fit = std::min(fit, (long long)256 * ROW_WAVES * (163840 / row_lds_bytes(bh)));
                const double r = (double)items / (double)fit;
                cost = (double)items * (bh + 2 * ROW_HX) * (t + 0.45 * xch) * (1.0 + 1.0 / r) * ((double)slots / (double)fit);
            } else {
                cost = row_time(bh, t + 0.15 * xch, (double)items, row_resident(slots, K, bh, diff));
            }
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = RowShape{bh, t};
            }
            if (req_h > 0) break;
        }
    }
    return best;
}

// How a frame-difference group of the Harris row kernel runs in a workspace with
// `room` bytes for its exchange: as planned where the words fit; else in the run
// (the planned one times a power of two) of least modelled time, each item
// recomputing the frame before its run where the words do not fit at that run
// either.  In the static 64 MiB, 640x480x1000 gray, planned at one frame a run,
// takes 587 us with two-frame runs (988 us recomputing at one), 800x600x700 RGB
// 728 us (1206 us).
struct RowRun {
    int tt, nchunks;
    bool exchange;
};
inline RowRun row_run(size_t room, int T, int nstrips, int nbands, int band_h, int K, int tt, int slots)
{
    RowRun best{};
    double best_time = -1.0;
    for (int t = tt;; t = t > T / 2 ? T : 2 * t) {
        const int n = (T + t - 1) / t;
        const bool fits = row_exchange_bytes(nstrips, nbands, n, band_h, K) <= room;
        const double time = row_time(band_h, t + (n == 1 ? 0.0 : fits ? 0.15 : 1.0), (double)nstrips * nbands * n,
                                     row_resident(slots, K, band_h, true));
        if (best_time < 0.0 || time < best_time) {
            best = RowRun{t, n, fits && n > 1};
            best_time = time;
        }
        if (fits) return best;  // n == 1 needs no words
    }
}

}  // namespace fz
