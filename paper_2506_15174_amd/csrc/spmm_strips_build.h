// Host builder of the strips path (format: spmm_strips.h); the one on the device (spmm_strips.hip) takes its units.
#ifndef SPMM_STRIPS_BUILD_H
#define SPMM_STRIPS_BUILD_H

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <numeric>
#include <vector>

#include "spmm_plan.h"
#include "spmm_strips.h"

namespace strips {

// Rows by length, longest first, stable; their lengths.
struct rows {
    std::vector<uint32_t> order, length;
};
inline rows by_length(int64_t M, const int32_t *row_ptr)
{
    int64_t longest = 0;
    for (int64_t i = 0; i < M; ++i) longest = std::max<int64_t>(longest, row_ptr[i + 1] - row_ptr[i]);
    rows r;
    r.order.resize((size_t)M);
    r.length.resize((size_t)M);
    if (longest < 8 * M + 4096) {  // counted
        std::vector<uint32_t> place((size_t)longest + 2, 0);
        for (int64_t i = 0; i < M; ++i) ++place[(size_t)(longest - (row_ptr[i + 1] - row_ptr[i])) + 1];
        for (size_t k = 1; k < place.size(); ++k) place[k] += place[k - 1];
        for (int64_t i = 0; i < M; ++i) {
            const uint32_t n = (uint32_t)(row_ptr[i + 1] - row_ptr[i]), at = place[(size_t)(longest - n)]++;
            r.order[at] = (uint32_t)i;
            r.length[at] = n;
        }
    } else {
        std::iota(r.order.begin(), r.order.end(), 0u);
        std::stable_sort(r.order.begin(), r.order.end(), [&](uint32_t x, uint32_t y) { return row_ptr[x + 1] - row_ptr[x] > row_ptr[y + 1] - row_ptr[y]; });
        for (int64_t i = 0; i < M; ++i) r.length[(size_t)i] = (uint32_t)(row_ptr[r.order[(size_t)i] + 1] - row_ptr[r.order[(size_t)i]]);
    }
    return r;
}

struct unit {
    int64_t first;  // place of its first row in the order
    int32_t parts_log2, steps;
};
constexpr int64_t steps_of(int64_t entries) { return (entries + STRIP_STEPS - 1) / STRIP_STEPS * STRIP_STEPS; }

// The rows in units whose lanes have at most `most` entries, where a row in 64 parts allows that.
inline void units_of(const rows &r, int64_t most, std::vector<unit> &units)
{
    units.clear();
    const int64_t M = (int64_t)r.length.size();
    units.reserve((size_t)(M / 8 + 64));
    int p = 6;
    for (int64_t at = 0; at < M;) {
        const int64_t len = r.length[(size_t)at];  // (no longer than those before)
        while (p > 0 && ((len + (1 << (p - 1)) - 1) >> (p - 1)) <= most) --p;
        units.push_back(unit{at, p, (int32_t)steps_of((len + (1 << p) - 1) >> p)});
        at += 64 >> p;
    }
}

inline void band_sizes(int64_t K, StripSizes &p)
{
    p.bands = (int32_t)((K + STRIP_MOST_ROWS - 1) / STRIP_MOST_ROWS);
    p.band_rows = (int32_t)(((K + p.bands - 1) / p.bands + STRIP_BAND_ALIGN - 1) / STRIP_BAND_ALIGN * STRIP_BAND_ALIGN);
}

// Columns of B that a plan without a hint is made for.
constexpr int64_t UNKNOWN_COLUMNS = 64;

// The units, longest first, for products with N columns, and their sizes (in bands: but for what bands leave idle): lanes of
// 0.8 to 1.6 equal shares of the entries, whichever is estimated to take least.  A row's parts are a power of two, so some
// shares leave some waves a second unit and others idle: with 1.25 shares for all 8968 x 2473, 92 % pruned, 96 columns takes
// 16.0 us instead of 14.0, 3001 x 2511, 85 %, 200 columns 18.4 instead of 17.8.  A strip in bands allows one unit per wave only,
// which more entries per lane bring about.
inline std::vector<unit> units_for(int64_t K, const rows &r, int64_t entries, int64_t N, StripSizes &p)
{
    band_sizes(K, p);
    const int64_t waves = STRIP_WAVES * std::max<int64_t>(1, 256 / ((N + STRIP_COLS - 1) / STRIP_COLS));  // with a workgroup on every compute unit
    std::vector<unit> best, units;
    StripSizes best_sizes = p;
    double best_us = 0.0;
    int64_t last_most = 0;
    for (const int64_t tenths : {8, 10, 12, 14, 16}) {
        int64_t most = std::max<int64_t>(8, steps_of(entries * tenths / (10 * 64 * waves) + 1));
        units_of(r, most, units);
        for (int tries = 0; p.bands > 1 && (int64_t)units.size() > waves && tries < 8; ++tries) {
            most += steps_of(most / 16 + 1);
            units_of(r, most, units);
        }
        if (most == last_most) continue;
        last_most = most;
        StripSizes s = p;
        s.n_units = (int64_t)units.size();
        for (const unit &u : units) {
            s.steps += u.steps;
            s.longest = std::max<int64_t>(s.longest, u.steps);
        }
        const double us = strip_time(s, K, N, nullptr);
        if (best.empty() || us < best_us) {
            best.swap(units);
            best_us = us;
            best_sizes = s;
        }
    }
    p = best_sizes;
    std::stable_sort(best.begin(), best.end(), [](const unit &x, const unit &y) { return x.steps > y.steps; });
    return best;
}

// Estimated time in us if no lane were idle and every wave had a unit: at hand without a look at the rows.
inline double time_at_best(int64_t M, int64_t K, int64_t entries, int64_t N)
{
    StripSizes p;
    band_sizes(K, p);
    p.n_units = std::max<int64_t>((M + 63) / 64, std::min<int64_t>(M, STRIP_WAVES * std::max<int64_t>(1, 256 / ((N + STRIP_COLS - 1) / STRIP_COLS))));
    p.steps = (entries + 63) / 64;
    return strip_time(p, K, N, nullptr);
}

// What strips have to beat where they were not asked for: the times of what a plan would hold instead, at some widths of B.
struct rivals {
    static constexpr int MOST = 5;
    int n = 0;
    int64_t N[MOST] = {};
    double us[MOST] = {};
    double crowding = 1.0;  // how much longer a step takes than the estimate says (look_at_columns)
    // Whether strips of these sizes are slower at one of the widths.
    bool faster_than(StripSizes p, int64_t K) const
    {
        p.steps = (int64_t)((double)p.steps * crowding);
        p.longest = (int64_t)((double)p.longest * crowding);
        for (int i = 0; i < n; ++i)
            if (strip_time(p, K, N[i], nullptr) > us[i]) return true;
        return false;
    }
    // The same of strips in bands when their steps have been counted.  A unit's lanes wait in every band for the fullest one,
    // which the rows' lengths do not tell: rows whose entries lie together leave most lanes idle in most bands.
    // Of 150 products that the lengths alone move (5100 to 16384 columns, rows even, lognormal or within a half, a third or a
    // quarter of the columns) the counted time is 1.00 of the measured one (rms 10 %), that of the others 0.90 of theirs.
    // From 1.1 times theirs on strips are left: 49 products, in which they take 1.12 times as long on average and up to 1.99
    // times; the 101 that stay take 0.73, 1.19 at worst.
    bool faster_than_counted(const StripSizes &p, int64_t K) const
    {
        rivals later = *this;
        for (double &t : later.us) t *= 1.1;
        return later.faster_than(p, K);
    }
};

// What a plan made for products with N columns begins with.
struct start {
    rows r;
    std::vector<unit> units;  // none: not looked at yet
    StripSizes sizes;
    rivals others;
    bool in_order = true;     // the columns of the rows that look_at_columns saw
    bool beaten = false;  // by them, when the strips in bands had been counted
};
inline void begin(int64_t M, int64_t K, const int32_t *row_ptr, int64_t N, start &s)
{
    if (!s.units.empty()) return;
    s.r = by_length(M, row_ptr);
    s.units = units_for(K, s.r, row_ptr[M], N, s.sizes);
}
inline int64_t columns_for(int32_t n_hint) { return n_hint > 0 ? n_hint : UNKNOWN_COLUMNS; }

// Words of the units and rows, in front of the groups.
inline size_t unit_words(int64_t n_units, int64_t bands) { return ((size_t)(n_units * bands) * 2 + (size_t)n_units * 64 + 63) / 64 * 64; }

inline void launches(StripPlan &p, int64_t K)
{
    for (int64_t s = 1; s <= StripPlan::KNOWN; ++s) {
        int64_t g = 0;
        strip_time(p, K, s * STRIP_COLS, &g);
        p.groups[s] = (uint32_t)g;
    }
}

struct host {
    StripPlan plan;  // without device memory
    raw_words stream;
    std::vector<uint32_t> units, rows;
};

// One thread's working memory.
struct scratch {
    std::vector<int32_t> order;
    std::vector<uint16_t> columns;  // of the unit's entries in the band, lane by lane, by column modulo 8
    std::vector<float> values;
};

// Orders and writes the entries of a unit in a band.  row_range(r, first, end): the r-th row's entries there, as places in `sorted`.
template <typename Row> void fill(const unit &u, int64_t n_rows, Row row_range, const int32_t *col_idx, const float *vals, const int32_t *sorted, int32_t band_first,
                                  uint32_t zero_row, int64_t groups, char *out, scratch &s)
{
    const int P = 1 << u.parts_log2;
    int32_t start[65], count[64][8], left[64];
    std::memset(count, 0, sizeof count);
    std::memset(left, 0, sizeof left);
    int64_t of_row[64][2];
    int32_t total = 0;
    for (int64_t r = 0; r < 64 / P; ++r) {
        of_row[r][0] = of_row[r][1] = 0;
        if (r < n_rows) row_range(r, of_row[r][0], of_row[r][1]);
        const int64_t n = of_row[r][1] - of_row[r][0];
        for (int x = 0; x < P; ++x) {
            start[r * P + x] = total;
            left[r * P + x] = (int32_t)((n + P - 1 - x) / P);
            total += left[r * P + x];
        }
    }
    s.columns.resize((size_t)total);
    s.values.resize((size_t)total);
    for (int64_t r = 0; r < 64 / P; ++r) {
        // the row's entries class by class (column modulo 8), dealt to its lanes in turn
        int32_t at[9] = {};
        for (int64_t q = of_row[r][0]; q < of_row[r][1]; ++q) ++at[((col_idx[sorted[q]] - band_first) & 7) + 1];
        for (int c = 1; c < 9; ++c) at[c] += at[c - 1];
        for (int64_t q = of_row[r][0]; q < of_row[r][1]; ++q) {
            const int32_t e = sorted[q], col = col_idx[e] - band_first, k = at[col & 7]++;
            const int lane = (int)(r * P + (k & (P - 1)));
            const size_t to = (size_t)(start[lane] + (k >> u.parts_log2));
            s.columns[to] = (uint16_t)col;
            s.values[to] = vals[e];
            ++count[lane][col & 7];
        }
    }
    const int32_t steps = (int32_t)(groups * STRIP_STEPS);
    for (int cycle = 0; cycle < 4; ++cycle) {
        int32_t total[2][8] = {}, most = 0;  // entries of a class that the even (odd) lanes hold
        for (int odd = 0; odd < 2; ++odd)
            for (int i = 0; i < 8; ++i)
                for (int c = 0; c < 8; ++c) most = std::max(most, total[odd][c] += count[strip_lane(cycle, i, odd)][c]);
        // where one class holds more entries than there are steps, it has to collide that often: in the same steps for all classes, even and odd
        const int32_t extra = std::max<int32_t>(0, most - steps);
        for (int odd = 0; odd < 2; ++odd) {
            int lanes[8];
            int32_t next[8][8];
            uint32_t has[8];  // classes
            for (int i = 0; i < 8; ++i) {
                const int l = lanes[i] = strip_lane(cycle, i, odd);
                int32_t to = start[l];
                has[i] = 0;
                for (int c = 0; c < 8; ++c) {
                    next[i][c] = to;
                    to += count[l][c];
                    has[i] |= (uint32_t)(count[l][c] > 0) << c;
                }
            }
            int32_t *sum = total[odd];
            uint32_t rich[8] = {}, above = 0;
            for (int32_t t = 0; t < steps; ++t) {
                const bool twice = extra >= steps || (int64_t)(t + 1) * extra / steps > (int64_t)t * extra / steps;
                if (t % STRIP_STEPS == 0) {  // classes of which a lane, all lanes hold more than of others
                    int32_t all = 0;
                    for (int c = 0; c < 8; ++c) all += sum[c];
                    above = 0;
                    for (int c = 0; c < 8; ++c) above |= (uint32_t)(sum[c] > all / 8) << c;
                    for (int i = 0; i < 8; ++i) {
                        rich[i] = 0;
                        for (int c = 0; c < 8; ++c) rich[i] |= (uint32_t)(count[lanes[i]][c] > left[lanes[i]] / 8) << c;
                    }
                }
                // Lane i takes class t + i if it has one.  Of the others each proposes a class, of those that are left and that it holds more of
                // if there is one, and of those that propose the same the first has it (in some steps: two have it); then once more.
                uint32_t once = 0, two = 0;  // classes that a lane took; that two did
                int take[8];
                for (int i = 0; i < 8; ++i) {
                    const int c = (t + i) & 7;
                    take[i] = has[i] >> c & 1 ? c : -1;
                    if (take[i] >= 0) once |= 1u << c;
                }
                for (const bool last : {false, true}) {
                    const uint32_t full = twice ? two : once;
                    for (int k = 0; k < 8; ++k) {
                        const int i = (t + k) & 7, from = (t + i) & 7;
                        if (take[i] >= 0) continue;
                        const bool waits = left[lanes[i]] < steps - t;  // it can (or it has none)
                        uint32_t can = has[i] & ~full;
                        if (!can) {
                            if (!last || waits) continue;
                            can = has[i];  // it collides
                        }
                        for (const uint32_t best : {rich[i] & above, rich[i], above})
                            if (can & best) {
                                can &= best;
                                break;
                            }
                        const int c = __builtin_ctz(can << 8 | (can >> from << from)) & 7;  // the first from t + i on, around
                        if ((twice ? two : once) >> c & 1 && !(last && !waits)) continue;
                        take[i] = c;
                        two |= once & 1u << c;
                        once |= 1u << c;
                    }
                }
                char *group = out + (size_t)(t / STRIP_STEPS) * STRIP_GROUP_BYTES;
                const int e = t % STRIP_STEPS;
                for (int i = 0; i < 8; ++i) {
                    const int l = lanes[i], c = take[i];
                    uint16_t place = (uint16_t)zero_row;
                    float value = 0.0f;
                    if (c >= 0) {
                        const size_t from = (size_t)next[i][c]++;
                        place = s.columns[from];
                        value = s.values[from];
                        --left[l];
                        --sum[c];
                        if (--count[l][c] == 0) has[i] &= ~(1u << c);
                    }
                    std::memcpy(group + l * 16 + e * 4, &value, 4);
                    std::memcpy(group + 1024 + l * 8 + e * 2, &place, 2);
                }
            }
        }
    }
}

constexpr int64_t MOST_GROUPS = 1 << 20;  // of a unit in a band (more take a column stored over and over in a row)

// over(n, job): job(first, end) over shares of n units, on several threads.  The columns have been checked.  False if A cannot be
// stored this way, or if what it has to beat is faster.
template <typename Over>
bool build(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, int64_t N, Over over, start &begun, host &out)
{
    out = host();
    if (M >= (int64_t)1 << STRIP_PARTS_SHIFT) return false;
    StripPlan &p = out.plan;
    begin(M, K, row_ptr, N, begun);
    const std::vector<uint32_t> &order = begun.r.order;
    const std::vector<unit> &units = begun.units;
    static_cast<StripSizes &>(p) = begun.sizes;
    const int64_t B = p.bands, R = p.band_rows;
    out.rows.resize((size_t)p.n_units * 64, STRIP_NO_ROW);
    out.units.resize((size_t)(p.n_units * B) * 2);
    std::vector<int64_t> groups((size_t)(p.n_units * B) + 1, 0);
    auto rows_of = [&](const unit &u) { return std::min<int64_t>(64 >> u.parts_log2, M - u.first); };
    // Places of a row's entries in order of the columns (stable), or null where they are stored in that order.
    auto canonical = [&](int64_t row, scratch &s) -> const int32_t * {
        const int32_t a = row_ptr[row], b = row_ptr[row + 1];
        bool sorted = true;
        for (int32_t q = a + 1; q < b && sorted; ++q) sorted = col_idx[q] >= col_idx[q - 1];
        if (sorted) return nullptr;
        s.order.resize((size_t)(b - a));
        std::iota(s.order.begin(), s.order.end(), a);
        std::stable_sort(s.order.begin(), s.order.end(), [&](int32_t x, int32_t y) { return col_idx[x] < col_idx[y]; });
        return s.order.data();
    };
    // ---- how many groups of steps every unit has in every band
    over(p.n_units, [&](int64_t first, int64_t end) {
        std::vector<int64_t> in_band((size_t)B);
        for (int64_t i = first; i < end; ++i) {
            const unit &u = units[(size_t)i];
            for (int64_t r = 0; r < rows_of(u); ++r) {
                const int64_t row = order[(size_t)(u.first + r)];
                for (int x = 0; x < 1 << u.parts_log2; ++x) out.rows[(size_t)(i * 64 + (r << u.parts_log2) + x)] = (uint32_t)row | (uint32_t)u.parts_log2 << STRIP_PARTS_SHIFT;
                if (B == 1) {
                    in_band[0] = row_ptr[row + 1] - row_ptr[row];
                } else {
                    std::fill(in_band.begin(), in_band.end(), (int64_t)0);
                    for (int32_t q = row_ptr[row]; q < row_ptr[row + 1]; ++q) ++in_band[(size_t)((uint32_t)col_idx[q] / (uint32_t)R)];
                }
                for (int64_t b = 0; b < B; ++b) {
                    int64_t &g = groups[(size_t)(i * B + b) + 1];
                    g = std::max(g, steps_of((in_band[(size_t)b] + (1 << u.parts_log2) - 1) >> u.parts_log2) / STRIP_STEPS);
                }
            }
        }
    });
    if (*std::max_element(groups.begin(), groups.end()) > MOST_GROUPS) return false;
    for (size_t k = 1; k < groups.size(); ++k) groups[k] += groups[k - 1];
    if (groups.back() >= (int64_t)1 << 32) return false;
    p.steps = groups.back() * STRIP_STEPS;
    p.longest = 0;
    for (int64_t i = 0; i < p.n_units; ++i) p.longest = std::max(p.longest, (groups[(size_t)((i + 1) * B)] - groups[(size_t)(i * B)]) * STRIP_STEPS);
    begun.beaten = B > 1 && begun.others.faster_than_counted(p, K);
    if (begun.beaten) return false;
    launches(p, K);
    for (int64_t k = 0; k < p.n_units * B; ++k) {
        out.units[(size_t)k * 2] = (uint32_t)groups[(size_t)k];
        out.units[(size_t)k * 2 + 1] = (uint32_t)(groups[(size_t)k + 1] - groups[(size_t)k]);
    }
    // ---- their entries
    out.stream.resize((size_t)groups.back() * (STRIP_GROUP_BYTES / 4));
    over(p.n_units, [&](int64_t first, int64_t end) {
        scratch s;
        std::vector<int32_t> sorted;      // the unit's rows in order of the columns
        std::vector<int64_t> begin(65);   // their places there
        for (int64_t i = first; i < end; ++i) {
            const unit &u = units[(size_t)i];
            const int64_t n = rows_of(u);
            sorted.clear();
            for (int64_t r = 0; r < n; ++r) {
                const int64_t row = order[(size_t)(u.first + r)];
                const int32_t *c = canonical(row, s);
                begin[(size_t)r] = (int64_t)sorted.size();
                if (c) sorted.insert(sorted.end(), c, c + (row_ptr[row + 1] - row_ptr[row]));
                else
                    for (int32_t q = row_ptr[row]; q < row_ptr[row + 1]; ++q) sorted.push_back(q);
            }
            begin[(size_t)n] = (int64_t)sorted.size();
            for (int64_t b = 0; b < B; ++b) {
                const int64_t band_first = b * R;
                auto range = [&](int64_t r, int64_t &from, int64_t &to) {
                    const auto lo = sorted.begin() + begin[(size_t)r], hi = sorted.begin() + begin[(size_t)r + 1];
                    auto before = [&](int64_t col) { return std::partition_point(lo, hi, [&](int32_t e) { return (int64_t)col_idx[e] < col; }) - sorted.begin(); };
                    from = B == 1 ? begin[(size_t)r] : before(band_first);
                    to = B == 1 ? begin[(size_t)r + 1] : before(band_first + R);
                };
                const size_t k = (size_t)(i * B + b);
                fill(u, n, range, col_idx, vals, sorted.data(), (int32_t)band_first, (uint32_t)R, groups[k + 1] - groups[k],
                     reinterpret_cast<char *>(out.stream.data()) + (size_t)groups[k] * STRIP_GROUP_BYTES, s);
            }
        }
    });
    return true;
}
template <typename Over> bool build(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, int64_t N, Over over, host &out)
{
    start begun;
    return build(M, K, row_ptr, col_idx, vals, N, over, begun, out);
}

}  // namespace strips

#endif
