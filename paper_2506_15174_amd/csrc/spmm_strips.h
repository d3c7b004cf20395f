// Strips path (internal): C in strips of eight columns, the strip of B in LDS, one lane per part of a row.
#ifndef SPMM_STRIPS_H
#define SPMM_STRIPS_H

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

// Format.  The rows are taken by length, longest first, in *units* of 64 lanes: a row is dealt to P lanes next to each
// other (its parts; P is a power of two, the same for all rows of a unit), so a unit holds 64 / P rows.  The columns of A are cut into
// `bands` of band_rows columns, one where the strip of B (32 bytes a row) fits LDS.  The entries of a unit in a band
// are stored in groups of four steps, a step being one entry of every lane:
//   values   64 x 16 bytes: the four values of lane 0, of lane 1, ...
//   places   64 x 8 bytes: their columns in the band, 16 bits each; band_rows (a row of zeros) where a lane has no entry
// The order of a lane's entries is free.  A wave reads 16 bytes of LDS for each of its lanes in four cycles, those
// of 16 lanes at a time (strip_lane names them), each cycle from 64 banks: even lanes read the first half of
// their rows of the strip, odd lanes the second, then the other one, so the eight even (odd) lanes of a cycle do not
// collide where their columns differ modulo 8.  The builder orders the entries by that.
constexpr int STRIP_COLS = 8, STRIP_ROW_BYTES = 4 * STRIP_COLS, STRIP_STEPS = 4, STRIP_GROUP_BYTES = 64 * (16 + 8);
constexpr int STRIP_LDS_BYTES = 160 * 1024, STRIP_BAND_ALIGN = 32;
constexpr int STRIP_MOST_ROWS = (STRIP_LDS_BYTES / STRIP_ROW_BYTES - 1) / STRIP_BAND_ALIGN * STRIP_BAND_ALIGN;  // of a band, but for the row of zeros
constexpr int STRIP_WAVES = 16;  // of a workgroup
// Lane i (0 .. 7) of the even (odd = 0) or odd ones among the 16 lanes that cycle `c` (0 .. 3) of a 16-byte read serves: lanes
// 0-3, 12-15, 20-23, 24-27, then 4-7, 8-11, 16-19, 28-31, then the same of the upper half (found by timing reads of which two
// lanes collide).
inline int strip_lane(int c, int i, int odd)
{
    constexpr int quads[2][4] = {{0, 12, 20, 24}, {4, 8, 16, 28}};
    return c / 2 * 32 + quads[c % 2][i / 2] + i % 2 * 2 + odd;
}

struct StripSizes {
    int64_t n_units = 0;            // 0 = the plan holds no strips
    // of all units, of one (as the rows' lengths tell, until the entries in every band have been counted)
    int64_t steps = 0, longest = 0;
    int32_t bands = 1, band_rows = 0;
};
struct StripPlan : StripSizes {
    static constexpr int KNOWN = 32;
    uint32_t groups[KNOWN + 1] = {};  // of units, for that many strips (strip_time)
    uint32_t *d_stream = nullptr;  // DEVICE groups, in the same memory behind
    // DEVICE per unit and band: first group, groups; behind them per unit and lane: row | log2(P) << 28, or STRIP_NO_ROW
    uint32_t *d_units = nullptr;  // (as many words as strips::unit_words, a multiple of 256 bytes)
    const uint32_t *d_rows() const { return d_units + n_units * bands * 2; }
    int64_t device_bytes = 0;
    bool built_on_device = false;  // whole, by spmm_strips_build_on_device
};
constexpr uint32_t STRIP_NO_ROW = 0xFFFFFFFFu;
constexpr int STRIP_PARTS_SHIFT = 28;

// Estimated time in us of a product with N columns of B, and the groups of units it runs with: a group is one workgroup
// per strip, and of one to eight rounds of 256 workgroups those are taken that take least.  (A wave has one unit
// at most where the strip comes in bands.)
// A workgroup's time: the copy of its strip (by the lines of 128 bytes that it touches; more where B exceeds an L2), its
// units' steps or, where those are few or uneven, its longest wave's, and the units' ends.
// Fitted to 420 products (256 to 16384 rows and columns, 2 to 50 % kept, 4 to 256 columns).  Of 420 others the rms error is
// 8.7 % (0.57 to 1.27 of the time back to back): 14 % below 8 columns, 7.5 % in one band, 11 % in several.
inline double strip_time(const StripSizes &p, int64_t K, int64_t N, int64_t *groups_out)
{
    const int64_t strips = (N + STRIP_COLS - 1) / STRIP_COLS, least = p.bands > 1 ? (p.n_units + STRIP_WAVES - 1) / STRIP_WAVES : 1;
    const double lines = std::min(1.0, (double)N / 32.0), beyond_l2 = std::min(1.0, std::max(0.0, 4e-6 / 4.2 * (double)K * (double)N - 0.75));
    const double copy = 1e-3 * (double)p.bands * p.band_rows * lines * (0.91 + 0.4 * beyond_l2), mean = (double)p.steps / (double)p.n_units;
    double best = 0.0;
    int64_t last = 0;
    for (int64_t r = 1; r <= 8; ++r) {
        const int64_t groups = std::min(p.n_units, std::max(least, 256 * r / strips)), rounds = (groups * strips + 255) / 256;
        if (groups == last) continue;
        last = groups;
        const double units = (double)p.n_units / (double)groups;
        const double all = 6.6e-3 * mean * units, wave = 40e-3 * std::max((double)p.longest, mean * std::ceil(units / STRIP_WAVES));
        const double us = (double)rounds * (2.7 + copy + 0.96 * (p.bands - 1) + std::sqrt(std::sqrt(all * all * all * all + wave * wave * wave * wave)) + 0.04 * units);
        if (best == 0.0 || us < best) {
            best = us;
            if (groups_out) *groups_out = groups;
        }
    }
    return best;
}

namespace strips {
struct start;
}
// Builds the strips of A on the current device from host CSR arrays whose row pointer has been checked; the columns are
// checked here.  N: the columns that the plan is for; begun: what it begins with, made here if it is empty.  Status codes
// follow spmm_status_t; STRIPS_NOT_POSSIBLE: a row's columns are not in order, a row has 65536 entries or more, there are more
// units than a launch takes, or steps than a plan, or what the strips have to beat is faster (begun.beaten).
constexpr int STRIPS_NOT_POSSIBLE = -1;
int spmm_strips_build_on_device(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, int64_t N,
                                strips::start &begun, StripPlan &out);
void spmm_strips_release(StripPlan &p);  // however it was built

// Strips of the first of the two sets in which a product's come, half of the XCDs fetching each; all: one set.
extern "C" uint32_t spmm_strips_of_set(int64_t steps, int64_t K, int32_t N);

// Enqueues C <- A x B.  Returns the hipError_t of the launch as int.
int spmm_strips_execute(const StripPlan &p, int64_t K, const float *B, int32_t N, float *C, void *stream);

#endif
