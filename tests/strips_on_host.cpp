// The strips that the builder makes (spmm_strips_build.h), read back as the kernel reads them: tests/test_strips_host.py
// compiles and runs this.  Every entry is found once, in a lane of its row, in the band of its column; what fills up names the row of zeros;
// and the lanes that read LDS together collide no more often than the builder's order is worth.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <tuple>

#include "spmm_strips_build.h"

#define REQUIRE(x) do { if (!(x)) { std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); std::exit(1); } } while (0)

struct csr {
    int64_t M, K;
    std::vector<int32_t> row_ptr{0}, col_idx;
    std::vector<float> vals;
};

// Rows of about `mean` entries, spread by `sigma`; every seventh empty; unsorted: any order, columns stored twice.
static csr matrix(int64_t M, int64_t K, double mean, double sigma, bool unsorted, unsigned seed)
{
    csr a{M, K};
    std::mt19937 g(seed);
    std::normal_distribution<double> z;
    for (int64_t i = 0; i < M; ++i) {
        int64_t n = i % 7 == 3 && M > 7 ? 0 : std::min<int64_t>(K, (int64_t)(mean * std::exp(sigma * z(g)) + 0.5));
        std::vector<int32_t> c;
        if (unsorted) {
            for (int64_t k = 0; k < n; ++k) c.push_back((int32_t)(g() % (uint64_t)K));
        } else {
            for (int64_t k = 0; k < K && n > 0; ++k)
                if ((int64_t)(g() % (uint64_t)(K - k)) < n) {
                    c.push_back((int32_t)k);
                    --n;
                }
        }
        for (int32_t k : c) {
            a.col_idx.push_back(k);
            a.vals.push_back((float)((int64_t)a.vals.size() + 1));  // each its own
        }
        a.row_ptr.push_back((int32_t)a.col_idx.size());
    }
    return a;
}

static strips::host made(const csr &a, int64_t N, int64_t share)
{
    strips::host h;
    auto over = [&](int64_t n, auto job) {
        for (int64_t i = 0; i < n; i += share) job(i, std::min(n, i + share));
    };
    REQUIRE(strips::build(a.M, a.K, a.row_ptr.data(), a.col_idx.data(), a.vals.data(), N, over, h));
    return h;
}

static double check(const csr &a, int64_t N)
{
    const strips::host h = made(a, N, 4);
    const StripPlan &p = h.plan;
    REQUIRE(p.n_units > 0 && p.bands * (int64_t)p.band_rows >= a.K && (p.band_rows + 1) * STRIP_ROW_BYTES <= STRIP_LDS_BYTES && p.band_rows % 32 == 0);
    REQUIRE((int64_t)h.rows.size() == p.n_units * 64 && (int64_t)h.units.size() == p.n_units * p.bands * 2);
    for (int64_t s = 1; s <= StripPlan::KNOWN; ++s) {  // a wave has one unit at most where the strip comes in bands
        REQUIRE(p.groups[s] >= 1 && p.groups[s] <= p.n_units);
        REQUIRE(p.bands == 1 || (int64_t)p.groups[s] * STRIP_WAVES >= p.n_units);
    }
    std::vector<int> lanes_of((size_t)a.M, 0);
    std::multimap<std::tuple<int64_t, int64_t>, float> found;
    int64_t steps = 0, next = 0, reads = 0, cycles = 0, longest = 0;
    for (int64_t u = 0; u < p.n_units; ++u) {
        const uint32_t log2 = h.rows[(size_t)u * 64] >> STRIP_PARTS_SHIFT;
        REQUIRE(h.rows[(size_t)u * 64] != STRIP_NO_ROW && log2 <= 6);  // the kernel takes the parts from lane 0
        int64_t of_unit = 0;
        for (int l = 0; l < 64; ++l) {
            const uint32_t w = h.rows[(size_t)u * 64 + l], first = h.rows[(size_t)u * 64 + (l >> log2 << log2)];
            REQUIRE(w == first && (w == STRIP_NO_ROW || w >> STRIP_PARTS_SHIFT == log2));
            if (w != STRIP_NO_ROW) ++lanes_of[(size_t)(w & ((1u << STRIP_PARTS_SHIFT) - 1))];
        }
        for (int64_t b = 0; b < p.bands; ++b) {
            const size_t k = (size_t)(u * p.bands + b) * 2;
            REQUIRE((int64_t)h.units[k] == next);
            next += h.units[k + 1];
            for (uint32_t g = 0; g < h.units[k + 1]; ++g) {
                const char *group = reinterpret_cast<const char *>(h.stream.data()) + (size_t)(h.units[k] + g) * STRIP_GROUP_BYTES;
                for (int e = 0; e < STRIP_STEPS; ++e) {
                    int use[4][2][8] = {}, place_of[64];
                    for (int l = 0; l < 64; ++l) {
                        uint16_t place;
                        float v;
                        std::memcpy(&v, group + l * 16 + e * 4, 4);
                        std::memcpy(&place, group + 1024 + l * 8 + e * 2, 2);
                        REQUIRE(place <= p.band_rows);
                        place_of[l] = place;
                        const uint32_t w = h.rows[(size_t)u * 64 + l];
                        if (place == p.band_rows) REQUIRE(v == 0.0f);
                        else found.emplace(std::make_tuple((int64_t)(w & ((1u << STRIP_PARTS_SHIFT) - 1)), b * p.band_rows + place), v);
                        REQUIRE(place == p.band_rows || w != STRIP_NO_ROW);
                    }
                    for (int c = 0; c < 4; ++c) {
                        int most = 1;
                        for (int odd = 0; odd < 2; ++odd)
                            for (int i = 0; i < 8; ++i) {
                                const int at = place_of[strip_lane(c, i, odd)];
                                if (at != p.band_rows) most = std::max(most, ++use[c][odd][at % 8]);
                            }
                        cycles += most;
                        ++reads;
                    }
                }
            }
            of_unit += h.units[k + 1] * STRIP_STEPS;
        }
        steps += of_unit;
        longest = std::max(longest, of_unit);
    }
    REQUIRE(steps == p.steps && next * STRIP_GROUP_BYTES == (int64_t)h.stream.size() * 4);
    REQUIRE(longest == p.longest);
    for (int64_t i = 0; i < a.M; ++i) REQUIRE(lanes_of[(size_t)i] > 0 && (lanes_of[(size_t)i] & (lanes_of[(size_t)i] - 1)) == 0);
    REQUIRE((int64_t)found.size() == (int64_t)a.vals.size());
    for (int64_t i = 0; i < a.M; ++i)
        for (int32_t q = a.row_ptr[(size_t)i]; q < a.row_ptr[(size_t)i + 1]; ++q) {
            const auto range = found.equal_range(std::make_tuple(i, (int64_t)a.col_idx[(size_t)q]));
            bool there = false;
            for (auto it = range.first; it != range.second; ++it) there |= it->second == a.vals[(size_t)q];
            REQUIRE(there);
        }
    // the same whatever the threads' shares
    const strips::host again = made(a, N, 1000);
    REQUIRE(again.stream.size() == h.stream.size() && again.units == h.units && again.rows == h.rows);
    REQUIRE(h.stream.empty() || std::memcmp(again.stream.data(), h.stream.data(), h.stream.size() * 4) == 0);
    return reads ? (double)cycles / (double)reads : 1.0;
}

int main()
{
    {   // every lane is served once
        std::vector<int> seen(64, 0);
        for (int c = 0; c < 4; ++c)
            for (int i = 0; i < 8; ++i)
                for (int odd = 0; odd < 2; ++odd) {
                    ++seen[(size_t)strip_lane(c, i, odd)];
                    REQUIRE(strip_lane(c, i, odd) % 2 == odd);
                }
        for (int n : seen) REQUIRE(n == 1);
    }
    unsigned seed = 0;
    for (bool unsorted : {false, true})
        for (int64_t N : {4, 64, 256})
            for (auto [M, K, mean, sigma] : {std::tuple<int64_t, int64_t, double, double>{1, 1, 1, 0}, {1, 5000, 5000, 0}, {3, 9, 4, 1}, {63, 64, 20, 0.5}, {64, 65, 3, 0},
                                             {65, 33, 40, 0}, {500, 700, 60, 1.5}, {2000, 40, 2, 1}, {130, STRIP_MOST_ROWS, 300, 0.5}, {130, STRIP_MOST_ROWS + 1, 300, 0.5},
                                             {300, 20000, 400, 1.5}, {1200, 6000, 20, 0.3}})
                check(matrix(M, K, mean, sigma, unsorted, ++seed), N);
    {   // no entry at all in some bands, in all
        csr a = matrix(100, 12000, 30, 0, false, 99);
        for (int32_t &c : a.col_idx) c = c % 3000 + 5200;
        check(a, 64);
        check(csr{5, 7, {0, 0, 0, 0, 0, 0}, {}, {}}, 64);
    }
    // Strips that were chosen, in bands, where the rows' entries lie together: a lane waits in every band for the fullest one, so
    // four bands take four times the steps that the rows' lengths tell, and what they have to beat is faster.
    for (int clustered = 0; clustered < 2; ++clustered) {
        csr a = matrix(2000, 16384, 1000, 0, false, 7);
        if (clustered)
            for (int64_t i = 0; i < a.M; ++i)
                for (int32_t q = a.row_ptr[(size_t)i]; q < a.row_ptr[(size_t)i + 1]; ++q) a.col_idx[(size_t)q] = (int32_t)(i * 7919 % 4 * 4096 + a.col_idx[(size_t)q] / 4);
        strips::start begun;
        strips::begin(a.M, a.K, a.row_ptr.data(), 128, begun);
        begun.others.n = 1;
        begun.others.N[0] = 128;
        begun.others.us[0] = 1.3 * strip_time(begun.sizes, a.K, 128, nullptr);
        strips::host h;
        const bool built = strips::build(a.M, a.K, a.row_ptr.data(), a.col_idx.data(), a.vals.data(), 128, [](int64_t n, auto job) { job(0, n); }, begun, h);
        std::printf("%s rows in bands: %lld steps counted, %lld by the rows' lengths\n", clustered ? "clustered" : "even", (long long)h.plan.steps, (long long)begun.sizes.steps);
        REQUIRE(built == !clustered && begun.beaten == (clustered == 1));
        begun.others.n = 0;  // asked for
        REQUIRE(strips::build(a.M, a.K, a.row_ptr.data(), a.col_idx.data(), a.vals.data(), 128, [](int64_t n, auto job) { job(0, n); }, begun, h) && !begun.beaten);
    }
    const double even = check(matrix(4096, 2048, 205, 0, false, 1000), 128);
    std::printf("collisions: %.3f cycles for one\n", even);
    REQUIRE(even < 1.3);  // at random 2.7
    std::printf("ok\n");
    return 0;
}
