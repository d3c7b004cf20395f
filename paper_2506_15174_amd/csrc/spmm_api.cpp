// C ABI of the library (include/spmm.h): plan life cycle, upload, execute-time
// dispatch of the gfx950 kernels.
#include "../../include/spmm.h"

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "spmm_format.h"
#include "spmm_kernels.h"
#include "spmm_plan.h"
#include "spmm_strips_build.h"
#include "spmm_tiles.h"

using namespace spmm_fmt;

struct spmm_plan {
    HostPlan host;
    bool on_device = false;
    int device = -1;
    uint32_t *d_stream = nullptr, *d_wins = nullptr, *d_items = nullptr, *d_rowmap = nullptr;
    // Panels cut across workgroups: one scratch slot of ufi x CROSS_ROW_FLOATS floats per
    // (column tile of a launch, workgroup of such a panel), written by every execute, and the
    // table of those panels.
    float *d_cross_sums = nullptr;
    uint32_t *d_cross_table = nullptr;
    // Plans cut along K: the slices' sums of one batch of up to KSLICE_COLS columns
    // (k_slices x slice_rows rows), written by every execute.
    float *d_slice_sums = nullptr;
    // tiles.rows > 0: the entries are in tiles and the product runs on the matrix cores; strips.n_units > 0: they are in
    // strips.  Otherwise they are in chunks.
    TilePlan tiles;
    StripPlan strips;
    bool on_chunks() const { return tiles.rows == 0 && strips.n_units == 0; }
    int64_t scratch_bytes = 0;
    int64_t device_bytes = 0;
    int64_t stream_words = 0;  // length of host.stream at creation (a device plan drops its host mirror)
    bool force_wide = false;  // spmm_options_t.force_wide: 64-bit addressing kernels also on small inputs
    int depth = 0;            // spmm_options_t.depth: pipeline depth asked for (0 = per-instance default)
    bool probe = false;       // spmm_options_t.probe: loads-only launches (measurement)
    int32_t heavy = 0;        // the first blocks that are heavier than most (heavy_blocks)
    int32_t n_dealt = 0;      // blocks behind the plan's own in d_items, dealt to the compute units (deal_blocks)
    // Whether 41 to 64, 97 to 119 and 120 to 128 columns run as two column tiles (spared_by_two_tiles)
    bool halved_64 = false, halved_119 = false, halved_128 = false;
};

namespace {

// Columns a plan cut along K computes per pair of launches (the width of its slices' buffer).
constexpr int32_t KSLICE_COLS = 128;

int64_t block_weight(const HostPlan &h, int64_t block)
{
    int64_t chunks = 0;
    for (int w = 0; w < WAVES_PER_WG; ++w) chunks += h.items[(size_t)((block * WAVES_PER_WG + w) * ITEM_WORDS + IT_NCHUNKS)];
    return chunks;
}

// The blocks up to the last of the first 256 that is half as heavy again as the mean.  (They come heaviest first, but for
// the order of split panels and whole ones.)
int32_t heavy_blocks(const HostPlan &h)
{
    int64_t last = std::min<int64_t>(h.n_blocks, 256);
    while (last > 0 && 2 * block_weight(h, last - 1) * h.n_blocks <= 3 * h.n_chunks) --last;
    return (int32_t)last;
}

// The blocks in the order in which compute units are loaded evenly; empty where the order they have does that.
//
// While all workgroups of a launch fit the chip the device deals them out in turn: block b goes to the unit of block
// b - 256 (looked up for 512 to 1024 workgroups of this size), whatever they weigh.  The blocks come heaviest first, so the
// first units get the heaviest of every round and, where the number of blocks is no multiple of 256, a block more.  Here every
// block, heaviest first, goes to the unit that has least so far, at most `per_unit` to one; a unit's r-th block is at place
// 256 r + unit, units with most blocks first, and idle blocks, which end at once, fill the places between.
// A gather is bound by the unit's vector L1, so a unit's time is the sum of its blocks' chunks; a block's start and end
// count as STARTING chunks.  A plan whose fullest unit gains less than 3 % keeps its order.
//
// In the plan's own order and dealt, lognormal rows, three plans and B in turn, us:
//   1024 x 4096, 90 % pruned, 64 columns, 552 blocks    10.0 -> 8.0
//   1024 x 2048, 90 %, 64 columns, 283 blocks            6.1 -> 5.2
//   1536 x 6144, 95 %, 64 columns, 644 blocks           10.3 -> 8.9
//   700 x 5000, 90 %, 100 columns, 321 of two rows      14.8 -> 13.1
//   2048 x 4096, 90 %, 32 columns, about 1000 blocks     8.6 -> 8.1
//   5000 x 2000, 97 %, 128 columns, 703 blocks           9.5 -> 8.8
// Twenty even, lognormal and Zipf matrices 8 % on average, none slower.  More blocks than the chip holds go to whichever unit is done first,
// and several column tiles have an order of their own (front_blocks).
std::vector<uint32_t> deal_blocks(const HostPlan &h, int per_unit)
{
    constexpr int64_t UNITS = 256, STARTING = 8;
    const int64_t n = h.n_blocks;
    if (n <= UNITS || n > UNITS * per_unit || h.k_slices > 1 || h.n_cross > 0) return {};
    std::vector<std::pair<int64_t, int32_t>> blocks((size_t)n);
    std::vector<int64_t> as_is((size_t)UNITS, 0);
    for (int64_t b = 0; b < n; ++b) {
        blocks[(size_t)b] = {block_weight(h, b) + STARTING, (int32_t)b};
        as_is[(size_t)(b % UNITS)] += blocks[(size_t)b].first;
    }
    std::stable_sort(blocks.begin(), blocks.end(), [](const auto &x, const auto &y) { return x.first > y.first; });
    struct unit {
        int64_t load;
        int32_t number;
        bool operator<(const unit &u) const { return load != u.load ? load > u.load : number > u.number; }  // the least loaded on top
    };
    std::vector<unit> heap((size_t)UNITS);
    std::vector<std::vector<int32_t>> of((size_t)UNITS);
    for (int32_t u = 0; u < UNITS; ++u) heap[(size_t)u] = {0, u};
    std::make_heap(heap.begin(), heap.end());
    int64_t most = 0;
    for (const auto &[weight, block] : blocks) {
        std::pop_heap(heap.begin(), heap.end());
        unit &u = heap.back();
        of[(size_t)u.number].push_back(block);
        u.load += weight;
        most = std::max(most, u.load);
        if ((int)of[(size_t)u.number].size() < per_unit) std::push_heap(heap.begin(), heap.end());
        else heap.pop_back();
    }
    if (most * 100 > *std::max_element(as_is.begin(), as_is.end()) * 97) return {};
    std::stable_sort(of.begin(), of.end(), [](const auto &x, const auto &y) { return x.size() > y.size(); });
    const int64_t rounds = (int64_t)of[0].size();
    int64_t last = 0;  // units with a block in the last round
    while (last < UNITS && (int64_t)of[(size_t)last].size() == rounds) ++last;
    constexpr size_t WORDS = (size_t)WAVES_PER_WG * ITEM_WORDS;
    std::vector<uint32_t> items((size_t)((rounds - 1) * UNITS + last) * WORDS, 0u);
    for (size_t at = 0; at < items.size(); at += WORDS) {
        const size_t place = at / WORDS, round = place / (size_t)UNITS;
        const std::vector<int32_t> &u = of[place % (size_t)UNITS];
        if (round < u.size()) std::copy_n(h.items.begin() + (ptrdiff_t)((size_t)u[round] * WORDS), WORDS, items.begin() + (ptrdiff_t)at);
        else for (size_t w = 0; w < (size_t)WAVES_PER_WG; ++w) items[at + w * ITEM_WORDS + IT_FLAGS] = FLAG_IDLE;
    }
    return items;
}

// What two column tiles spare the fullest compute unit of a launch of N columns in one tile of 64 or 128, in chunks (one is 64 cycles of
// the vector L1); 0 where that is not worth it.
//
// A launch of up to 512 blocks ends with its fullest unit.  Of up to 128 blocks a block's two tiles, each about half of its time, go to two units of
// which one would be idle; of more, even ones too, a unit with a block more than another or a heavy one gets half a block there.  Against that, two
// tiles read the plan twice and have twice the starts and ends, about 0.3 us, and where rows of B are no whole lines they fetch more lines.
// The loads of both launches are counted in the order in which their workgroups start (front_blocks: block by block from 120 columns on, below at most
// the heavy ones or 128 first); blocks as in deal_blocks.  us in one tile and in two, plans and B in turn, and what the fullest unit is spared:
//   1103 x 7373, 99 %, Zipf, 97 columns        34.4 and 19.0   248 of 511     506 x 902, 94 %, Zipf, 97              5.75 and 4.41   64 of 127
//   300 x 4096, 90 % lognormal, 128            11.0 and 7.1     65 of 192     512 x 2048, 90 % lognormal, 128        6.08 and 5.51   36 of 125
//   2048 x 2048, 98 %, Zipf, 128                8.6 and 6.5     68 of 192     365 x 2494, 98 % lognormal, 128        3.34 and 3.10   20 of 40
//   512 x 512, 80 %, 128                       3.62 and 3.97    12 of 63      424 x 2254, 94 %, 100                  4.02 and 4.79   -5 of 63
//   512 x 2048, 90 %, 128                      5.02 and 5.10     4 of 69      6837 x 1529, 99 %, Zipf, 97 (1131 blocks)  6.3 and 9.2  21 of 168
// A chunk's rows of B in tiles of 64 and 32 columns take half the time, and four slices and eight more of the rest:
//   566 x 14392, 98 %, Zipf, 64 columns        47.6 and 26.3   904 of 1808    1256 x 5508, 98 %, Zipf, 56            18.0 and 12.6  320 of 656
//   958 x 3397, 98 %, Zipf, 48                 6.51 and 6.15   124 of 264     1971 x 3239, 98 %, Zipf, 64            6.77 and 6.64  120 of 280
//   541 x 8687, 90 % lognormal, 56             14.0 and 14.2   110 of 413     992 x 1742, 98 %, Zipf, 48             4.09 and 4.25   44 of 104
// 183 chunk plans of 64 to 4096 rows, Zipf, lognormal and even: at 120 to 128 columns 28 are taken (20 chunks, a sixth of the load), 1.21 times as fast on
// average and 1 % slower at worst; at 97 to 119 39, 1.16 times and 1 % at worst; at 41 to 64 (120 chunks) 33, 1.19 times and none slower.  Taller panels, whose chunks are
// multiplied by more rows, below 120 columns only for a quarter: 657 x 7119, 95 % lognormal, 119 columns 13.2 and 14.4 (46 of 265), 815 x 3535,
// 96 %, 119, 8.1 and 8.6 (31 of 163).  With the loads counted as if all launches went block by block 14 of 54 at 97 to 119 columns were slower, up to 11 %.
int64_t spared_by_two_tiles(const HostPlan &h, const std::vector<uint32_t> &dealt, int32_t heavy, int32_t N)
{
    constexpr int64_t UNITS = 256, STARTING = 8;
    if (h.ufk != UFK || h.n_blocks > 2 * UNITS || h.k_slices > 1 || h.n_cross > 0) return 0;
    constexpr size_t WORDS = (size_t)WAVES_PER_WG * ITEM_WORDS;
    spmm_launch_args a;
    a.width = N;
    a.heavy = heavy;
    auto fullest = [&](const std::vector<uint32_t> &items, int32_t tiles, int32_t tile_cols) {
        a.n_blocks = (int32_t)(items.size() / WORDS);
        a.n_tiles = tiles;
        a.tile_cols = tile_cols;
        const launch_shape shape{(uint32_t)a.n_blocks, (uint32_t)tiles, front_blocks(a)};
        std::vector<int64_t> load((size_t)UNITS, 0);
        for (uint32_t y = 0; y < shape.n_tiles; ++y)
            for (uint32_t x = 0; x < shape.n_blocks; ++x) {
                const uint32_t *block = items.data() + place_of(shape, launch_group{x, y}).block * WORDS;
                int64_t chunks = 0;
                for (int w = 0; w < WAVES_PER_WG; ++w) chunks += block[w * ITEM_WORDS + IT_NCHUNKS];
                if (chunks > 0) load[(y * shape.n_blocks + x) % (uint32_t)UNITS] += chunks + STARTING;
            }
        return *std::max_element(load.begin(), load.end()) / tiles;
    };
    const int32_t half = N > 64 ? 64 : 32;
    const int64_t one = fullest(dealt.empty() ? h.items : dealt, 1, 2 * half), spared = one - fullest(h.items, 2, half);
    return spared >= (N > 64 ? 20 : 120) && spared * (h.ufi > 1 && N < 120 ? 4 : 6) >= one ? spared : 0;
}

spmm_status_t hip_fail()
{
    (void)hipGetLastError();  // clear the sticky error
    return SPMM_ERR_HIP;
}

template <typename T>
spmm_status_t upload(T **dst, const void *src, size_t bytes, int64_t &total)
{
    *dst = nullptr;
    if (bytes == 0) return SPMM_OK;
    void *p = nullptr;
    hipError_t e = hipMalloc(&p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e == hipErrorOutOfMemory ? SPMM_ERR_ALLOC : SPMM_ERR_HIP;
    }
    *dst = static_cast<T *>(p);
    total += (int64_t)bytes;
    if (src) {
        if (hipMemcpy(p, src, bytes, hipMemcpyHostToDevice) != hipSuccess) return hip_fail();
    } else {
        if (hipMemset(p, 0, bytes) != hipSuccess) return hip_fail();
    }
    return SPMM_OK;
}

// Whether the arrays can be handed to a device: dimensions, pointers and the row pointer
// (the inspector, which checks the same, names the fault of arrays that cannot).
bool row_pointer_ok(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals)
{
    if (M <= 0 || K <= 0 || M > INT32_MAX || K > INT32_MAX || !row_ptr || row_ptr[0] != 0 || !col_idx || !vals) return false;
    for (int64_t i = 0; i < M; ++i)
        if (row_ptr[i + 1] < row_ptr[i]) return false;
    return true;
}

// Strips that the host builds, from rows in any order.  SPMM_OK and no units: A cannot be stored this way, or there is no room for
// it, on the host or on the device; chunks need less of both.
spmm_status_t strips_from_host(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals,
                               const InspectorOptions &io, strips::start &begun, StripPlan &out)
{
    strips::host made;
    try {
        const int rc = spmm_strips_build(M, K, row_ptr, col_idx, vals, io.n_hint, io.threads, begun, made);
        if (rc != 0) return (spmm_status_t)rc;
    } catch (const std::bad_alloc &) {
        return SPMM_OK;
    }
    if (made.plan.n_units == 0) return SPMM_OK;
    const size_t front = strips::unit_words(made.plan.n_units, made.plan.bands), bytes = (front + made.stream.size()) * 4;
    void *memory = nullptr;
    const hipError_t e = hipMalloc(&memory, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e == hipErrorOutOfMemory ? SPMM_OK : SPMM_ERR_HIP;
    }
    out = made.plan;  // its owner releases the memory
    out.d_units = static_cast<uint32_t *>(memory);
    out.d_stream = out.d_units + front;
    out.device_bytes = (int64_t)bytes;
    auto copy = [](uint32_t *to, const auto &words) { return words.empty() || hipMemcpy(to, words.data(), words.size() * 4, hipMemcpyHostToDevice) == hipSuccess; };
    return copy(out.d_units, made.units) && copy(out.d_units + made.units.size(), made.rows) && copy(out.d_stream, made.stream) ? SPMM_OK : hip_fail();
}

struct plan_release {
    void operator()(spmm_plan *p) const
    {
        bool held = p->tiles.rows > 0 || p->strips.d_units;
        for (void *q : {(void *)p->d_stream, (void *)p->d_wins, (void *)p->d_items, (void *)p->d_rowmap, (void *)p->d_cross_sums,
                        (void *)p->d_cross_table, (void *)p->d_slice_sums})
            if (q) {
                held = true;
                (void)hipFree(q);
            }
        spmm_tiles_release(p->tiles);
        spmm_strips_release(p->strips);
        if (held) (void)hipGetLastError();
        delete p;
    }
};
typedef std::unique_ptr<spmm_plan, plan_release> plan_owner;

// spmm_plan_create_sized but for the exceptions of the host containers, which its caller turns into a status.
spmm_status_t create(plan_owner &plan, int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx,
                     const float *vals, const spmm_options_t &opts)
{
    InspectorOptions io;
    bool host_only = false, force_wide = false, probe = false, schedule_forced = false;
    int depth = 0, tiles = 0;
    if (opts.group_nnz < 0 || opts.group_panels < 0 || opts.n_hint < 0) return SPMM_ERR_INVALID_ARG;
    if (opts.ufi != 0 && opts.ufi != 1 && opts.ufi != 2 && opts.ufi != 4 && opts.ufi != 8)
        return SPMM_ERR_INVALID_ARG;
    if (opts.threads < 0 || opts.threads > 64) return SPMM_ERR_INVALID_ARG;
    if (opts.depth != 0 && opts.depth != 1 && opts.depth != 2 && opts.depth != 3 && opts.depth != 4 &&
        opts.depth != 8)
        return SPMM_ERR_INVALID_ARG;
    io.ufi = opts.ufi;
    io.group_nnz = opts.group_nnz;
    io.group_panels = opts.group_panels;
    host_only = opts.host_only != 0;
    io.n_hint = opts.n_hint;
    io.sort_rows = opts.sort_rows;
    io.threads = opts.threads;
    io.cross = opts.cross;
    if (opts.kslices != 0 && opts.kslices != 1 && opts.kslices != 2 && opts.kslices != 4 && opts.kslices != 8)
        return SPMM_ERR_INVALID_ARG;
    io.kslices = opts.kslices;
    if (opts.ufk != 0 && !valid_ufk(opts.ufk)) return SPMM_ERR_INVALID_ARG;
    io.ufk = opts.ufk;
    force_wide = opts.force_wide != 0;
    if (force_wide) io.ufk = UFK;  // the 64-bit addressing kernels read chunks of 8 columns
    if (io.kslices > 1 && io.ufk != 0 && io.ufk != UFK) return SPMM_ERR_INVALID_ARG;  // only plans with chunks of 8 are cut
    depth = opts.depth;
    probe = opts.probe != 0;
    if (opts.tiles > 0 && opts.tiles != 8 && opts.tiles != 16 && opts.tiles != 32) return SPMM_ERR_INVALID_ARG;
    tiles = opts.tiles;
    // settings of the chunk path ask for the chunk path
    schedule_forced = opts.ufi || opts.group_nnz || opts.group_panels || opts.sort_rows || force_wide || depth || opts.cross ||
                      opts.ufk || probe || opts.kslices;
    if (probe && (force_wide || depth != 0 || (io.ufk != 0 && io.ufk > 16))) return SPMM_ERR_INVALID_ARG;
    plan.reset(new spmm_plan());
    spmm_plan *p = plan.get();
    int rc = 0;
    bool use_strips = opts.strips > 0 && tiles <= 0;
    if (use_strips && (schedule_forced || host_only)) return SPMM_ERR_INVALID_ARG;
    const bool checked = row_pointer_ok(M, K, row_ptr, col_idx, vals);
    strips::start begun;
    int32_t instead = 0;  // tiles that strips take the place of
    if (!host_only && tiles == 0 && !use_strips && !schedule_forced && checked) {
        chunk_estimate chunks;
        tiles = choose_tiles(M, K, row_ptr, io.n_hint, chunks);
        if (opts.strips == 0 && choose_strips(M, K, row_ptr, col_idx, io.n_hint, tiles, chunks, begun)) {
            use_strips = true;
            instead = tiles;
            tiles = 0;
        }
    }
    if (use_strips && checked && row_ptr[M] > 0) {
        if (opts.strips > 0) look_at_columns(M, row_ptr, col_idx, begun);
        rc = begun.in_order ? spmm_strips_build_on_device(M, K, row_ptr, col_idx, vals, strips::columns_for(io.n_hint), begun, p->strips)
                            : STRIPS_NOT_POSSIBLE;
        if (rc == STRIPS_NOT_POSSIBLE || rc == SPMM_ERR_ALLOC) {
            rc = 0;
            if (instead > 0) tiles = instead;  // which the device builds from rows in any order
            else if (!begun.beaten) rc = strips_from_host(M, K, row_ptr, col_idx, vals, io, begun, p->strips);
        }
        io.schedule_only = p->strips.n_units > 0;
    }
    if (rc == 0 && !host_only && tiles > 0 && checked) {
        rc = spmm_tiles_build(M, K, row_ptr, col_idx, vals, tiles, p->tiles);
        // the chunk plan needs no memory beside its own, the builder of tiles a multiple of its result's
        if (rc == TILES_NOT_POSSIBLE || rc == SPMM_ERR_ALLOC) rc = 0;
        io.schedule_only = p->tiles.rows > 0;
    }
    if (rc == 0) rc = spmm_inspect(M, K, row_ptr, col_idx, vals, io, p->host);
    if (rc != 0) return (spmm_status_t)rc;
    p->force_wide = force_wide;
    p->depth = depth;
    p->probe = probe;
    if (!host_only) {
        if (hipGetDevice(&p->device) != hipSuccess) return hip_fail();
        const HostPlan &h = p->host;
        spmm_status_t st = SPMM_OK;
        if (!p->on_chunks()) {
            p->device_bytes = p->tiles.device_bytes + p->strips.device_bytes;
        } else {
            // Scratch first: hipMemset may return before it is done, the copies behind it do not.
            if (h.n_cross_slots > 0) {
                const size_t slots = (size_t)h.n_cross_slots * CROSS_MAX_TILES;
                st = upload(&p->d_cross_sums, nullptr, slots * (size_t)h.ufi * CROSS_ROW_FLOATS * sizeof(float), p->device_bytes);
                // set-up for spmm_execute_static: this device's address of the static scratch is looked up here,
                // once, so that the entry point itself finds it ready (a failure only matters to that entry point)
                float *unused = nullptr;
                size_t unused_bytes = 0;
                if (spmm_static_scratch(&unused, &unused_bytes) != 0) (void)hipGetLastError();
            }
            if (st == SPMM_OK && h.k_slices > 1)
                st = upload(&p->d_slice_sums, nullptr, (size_t)h.plan_rows * KSLICE_COLS * sizeof(float), p->device_bytes);
            p->scratch_bytes = p->device_bytes;
            if (st == SPMM_OK) st = upload(&p->d_rowmap, h.rowmap.data(), h.rowmap.size() * 4, p->device_bytes);
            if (st == SPMM_OK) st = upload(&p->d_cross_table, h.cross.data(), h.cross.size() * 4, p->device_bytes);
            if (st == SPMM_OK) st = upload(&p->d_stream, h.stream.data(), h.stream.size() * 4, p->device_bytes);
            if (st == SPMM_OK) st = upload(&p->d_wins, h.wins.data(), h.wins.size() * 4, p->device_bytes);
            p->heavy = heavy_blocks(h);
            // for the widest tile of as many columns as the plan is meant for
            const int slices = h.ufk == 16 ? 8 : h.ufk == 32 ? 16 : h.ufk == 64 ? 32 : io.n_hint <= 0 || io.n_hint > 64 ? 2 : io.n_hint > 32 ? 4 : 8;
            std::vector<uint32_t> dealt = deal_blocks(h, workgroups_per_unit(slices, h.ufi, h.ufk, false));
            p->n_dealt = (int32_t)(dealt.size() / ((size_t)WAVES_PER_WG * ITEM_WORDS));
            p->halved_64 = spared_by_two_tiles(h, dealt, p->heavy, 64) > 0;
            p->halved_119 = spared_by_two_tiles(h, dealt, p->heavy, 119) > 0;
            p->halved_128 = spared_by_two_tiles(h, dealt, p->heavy, 128) > 0;
            if (p->n_dealt > 0) dealt.insert(dealt.begin(), h.items.begin(), h.items.end());
            const std::vector<uint32_t> &items = p->n_dealt > 0 ? dealt : h.items;
            if (st == SPMM_OK) st = upload(&p->d_items, items.data(), items.size() * 4, p->device_bytes);
        }
        if (st != SPMM_OK) return st;
        p->on_device = true;
    }
    const StripPlan &on_strips = p->strips;
    p->stream_words = p->tiles.rows > 0          ? p->tiles.stream_words
                      : on_strips.n_units > 0    ? on_strips.steps / STRIP_STEPS * (STRIP_GROUP_BYTES / 4)
                                                 : (int64_t)p->host.stream.size();
    if (on_strips.n_units > 0) {
        p->host.n_enum = on_strips.steps * 64;
        p->host.n_chunks = on_strips.n_units * on_strips.bands;
    }
    if (p->tiles.rows > 0) {
        p->host.n_enum = p->tiles.n_panels * K;
        p->host.n_chunks = p->tiles.n_panels * p->tiles.n_steps;
    }
    if (p->on_device) {
        // the arrays live on the device now: keep the descriptors (row groups, sizes), not the mirror
        raw_words().swap(p->host.stream);
        std::vector<uint32_t>().swap(p->host.hdr);
        std::vector<uint32_t>().swap(p->host.wins);
        std::vector<uint32_t>().swap(p->host.items);
        // the row map stays: one bit of it (sorted or not) is part of the description
    }
    return SPMM_OK;
}

}  // namespace

extern "C" {

spmm_status_t spmm_plan_create_sized(spmm_plan_t **plan, int64_t M, int64_t K, const int32_t *row_ptr,
                                     const int32_t *col_idx, const float *vals, const spmm_options_t *opts,
                                     size_t opts_bytes)
{
    if (!plan) return SPMM_ERR_INVALID_ARG;
    *plan = nullptr;
    spmm_options_t known;
    std::memset(&known, 0, sizeof known);
    if (opts) {
        std::memcpy(&known, opts, std::min(opts_bytes, sizeof known));
        for (size_t i = sizeof known; i < opts_bytes; ++i)
            if (reinterpret_cast<const unsigned char *>(opts)[i]) return SPMM_ERR_UNSUPPORTED;
    }
    try {
        plan_owner made;  // gives back what it holds unless it is handed over
        const spmm_status_t st = create(made, M, K, row_ptr, col_idx, vals, known);
        if (st == SPMM_OK) *plan = made.release();
        return st;
    } catch (const std::bad_alloc &) {
        return SPMM_ERR_ALLOC;
    } catch (...) {  // length errors of the containers and the like
        return SPMM_ERR_UNSUPPORTED;
    }
}

spmm_status_t spmm_plan_create(spmm_plan_t **plan, int64_t M, int64_t K, const int32_t *row_ptr,
                               const int32_t *col_idx, const float *vals)
{
    return spmm_plan_create_sized(plan, M, K, row_ptr, col_idx, vals, nullptr, 0);
}

spmm_status_t(spmm_plan_create_ex)(spmm_plan_t **plan, int64_t M, int64_t K, const int32_t *row_ptr,
                                   const int32_t *col_idx, const float *vals, const spmm_options_t *opts)
{
    return spmm_plan_create_sized(plan, M, K, row_ptr, col_idx, vals, opts, offsetof(spmm_options_t, tiles));
}

namespace {

// How a plan's chunks take N columns of B.
struct column_tiles {
    bool wide, quads, sliced, narrow_tiles, three_tiles, two_tiles;
    int ufk;
    int32_t N;

    column_tiles(const spmm_plan &plan, int32_t n) : ufk(plan.host.ufk), N(n)
    {
        const HostPlan &h = plan.host;
        const uint64_t b_total = (uint64_t)h.K * (uint64_t)N * 4u;
        // Narrow addressing: 32-bit byte offsets into B formed by a 24 x 24-bit multiply.
        const bool narrow_ok = b_total <= 0xFFFFFFFFull && h.K < (1 << 24) && (uint64_t)N * 4u < (1u << 24);
        wide = !narrow_ok || (plan.force_wide && b_total > 0);
        // Four columns per lane: 16-byte loads and stores at 4-byte alignment are legal, and a
        // last lane with fewer than four columns reads past the end of its rows of B, which is
        // safe through the buffer descriptor of the narrow addressing only (range-checked).
        quads = !wide || N % 4 == 0;
        sliced = h.k_slices > 1;
        // A 128-column tile of B that exceeds one L2 (4 MiB) while a 64-column tile fits: two
        // narrower tiles read the plan twice but keep their rows of B L2-resident (measured on a
        // 16384-column matrix of 13 M nonzeros: 275 against 295 us).
        // (A plan cut along K binds every slice of B to the L2s of its own XCDs instead and runs full tiles.)
        narrow_tiles = !sliced && (int64_t)h.K * 512 > ((int64_t)4 << 20) && (int64_t)h.K * 256 <= ((int64_t)4 << 20);
        // 161 to 192 columns are three tiles of 64 in one launch: as 128 and 64 the launch of the wide tile drains
        // before that of the rest begins.  24 even and uneven matrices at 161, 176, 188 and 192 columns: 13 to 18 % faster on
        // average, 2 % slower at worst (24 others 12 to 17 and 6 %).  Single
        // rows share no load, and a row of B that begins inside of a cache line takes one line in three more than its
        // columns in tiles of 64, one in five in tiles of 128: from 2^19 entries on even ones are up to 11 % slower then, uneven ones
        // between 14 % faster and 9 % slower; below, up to twice as fast.
        // 129 to 160 columns, 128 and a tile of 32, stay: as three tiles of 64 the 24 matrices are 5 % slower on average at 130 columns, 1 % at 144 and 3 % faster at 160
        // (0.75 to 1.24 of the time).
        three_tiles = !sliced && !wide && ufk == UFK && N > 160 && N <= 192 && (h.ufi > 1 || (N % 32 == 0 && plan.heavy == 0) || h.nnz < ((int64_t)1 << 19));
        two_tiles = !wide && (N > 96 ? N < 120 ? plan.halved_119 : N <= 128 && plan.halved_128 : N > 40 && N <= 64 && plan.halved_64);
    }
    // Columns of a tile where `left` are to be computed, and its slices.
    int32_t tile_for(int32_t left, int &slices) const
    {
        if (ufk != UFK) {
            slices = ufk == 16 ? 8 : ufk == 32 ? 16 : left > 4 ? 32 : 64;
            return 256 / slices;
        }
        if (!quads) {
            slices = 1;
            return 64;
        }
        slices = left > 64 ? (narrow_tiles || three_tiles || two_tiles ? 4 : 2) : left > 32 && !(two_tiles && N <= 64) ? 4 : 8;
        return 256 / slices;
    }
    // The next launch of those: its tiles, their columns (the last may have fewer) and slices, and the columns of all.
    int32_t launch(int32_t left, int32_t &tile, int32_t &cols, int &slices) const
    {
        tile = tile_for(left, slices);
        const int32_t n_tiles = left / tile;
        cols = n_tiles * tile;
        int rest_slices = 0;
        if (n_tiles == 0 || (left > cols && tile_for(left - cols, rest_slices) == tile)) {
            cols = left;  // the narrower last tile runs on the same kernel
            return n_tiles + 1;
        }
        return n_tiles;
    }
};

// cross_sums: scratch for the sums of panels cut across workgroups, with room for
// cross_tiles column tiles of one launch (unused by plans without such panels)
spmm_status_t execute_with(const spmm_plan_t *plan, const float *B, int32_t N, float *C, void *stream,
                           float *cross_sums, int32_t cross_tiles)
{
    if (!plan || N < 1) return SPMM_ERR_INVALID_ARG;
    if (!plan->on_device) return SPMM_ERR_INVALID_ARG;
    const HostPlan &h = plan->host;
    if (h.M == 0) return SPMM_OK;
    if (!C) return SPMM_ERR_INVALID_ARG;
    if (h.K > 0 && !B) return SPMM_ERR_INVALID_ARG;
    if (((uintptr_t)B & 3u) || ((uintptr_t)C & 3u)) return SPMM_ERR_INVALID_ARG;
    // the plan's arrays live on the device that was current when it was created
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return hip_fail();
    if (dev != plan->device) return SPMM_ERR_INVALID_ARG;

    if (plan->strips.n_units > 0) return spmm_strips_execute(plan->strips, h.K, B, N, C, stream) == 0 ? SPMM_OK : hip_fail();
    if (plan->tiles.rows > 0) return spmm_tiles_execute(plan->tiles, h.M, h.K, B, N, C, stream) == 0 ? SPMM_OK : hip_fail();

    const column_tiles tiling(*plan, N);
    const bool wide = tiling.wide, sliced = tiling.sliced;
    const uint64_t b_total = (uint64_t)h.K * (uint64_t)N * 4u;
    spmm_launch_args a;
    a.stream = plan->d_stream;
    a.wins = plan->d_wins;
    a.items = plan->d_items;
    a.rowmap = plan->d_rowmap;
    a.n_blocks = (int32_t)h.n_blocks;
    a.ldn = N;
    a.ldc = N;
    a.k_slices = h.k_slices;
    a.slice_rows = h.slice_rows;
    a.M = h.M;
    a.col_mask = h.K <= ((int64_t)1 << spmm_fmt::COL_PATTERN_SHIFT) ? spmm_fmt::COL_INDEX_MASK : 0xFFFFFFFFu;
    a.cross_sums = cross_sums;
    a.cross_table = plan->d_cross_table;
    a.n_cross_slots = (uint32_t)h.n_cross_slots;
    a.n_cross = (int32_t)h.n_cross;
    a.heavy = plan->heavy;
    a.probe = plan->probe;
    if (plan->probe && (wide || h.ufk > 16)) return SPMM_ERR_UNSUPPORTED;
    // the scratch of panels cut across workgroups holds so many column tiles of one launch
    const int32_t max_tiles = sliced ? 1 : h.n_cross_slots > 0 ? cross_tiles : 65535;
    // A tile of 64 columns where 128 exceed the L2 fills it: two workgroups per CU instead of three keep the
    // rows of B that concurrently running waves sweep inside it (16384 columns, 13 M nonzeros: 262 against 275 us).
    const uint32_t tile_pad = tiling.narrow_tiles ? 24u << 10 : 0u;
    // Column tiles of one width share a launch (front_blocks: in which order; a
    // tile begins while the previous one drains); a narrower rest takes a launch of its own.
    // Plans made for narrow B (chunks wider than 8 columns) run every N on their own narrow tiles.
    if (h.ufk != UFK && wide) return SPMM_ERR_UNSUPPORTED;
    int32_t j0 = 0;
    while (j0 < N) {
        // a plan cut along K takes the columns in batches its slices' buffer holds
        const int32_t left = sliced && N - j0 > KSLICE_COLS ? KSLICE_COLS : N - j0;
        int slices = 0;
        int32_t tile = 0, cols = 0, n_tiles = tiling.launch(left, tile, cols, slices);
        if (n_tiles > max_tiles) {  // grid limit, or the scratch's; the loop takes the rest
            n_tiles = max_tiles;
            cols = n_tiles * tile;
        }
        a.B = B ? B + j0 : nullptr;
        a.C = C + j0;
        if (sliced) {
            // the launch writes the slices' sums, rows of (cols rounded up to 4) floats; its
            // last step adds them into C
            a.C = plan->d_slice_sums;
            a.ldc = (cols + 3) / 4 * 4;
            a.C_out = C + j0;
            a.ldc_out = N;
        }
        a.width = cols;
        a.tile_cols = tile;
        a.n_tiles = n_tiles;
        a.lds_pad = tile_pad;
        const bool dealt = n_tiles == 1 && tile_pad == 0 && plan->n_dealt <= 256 * workgroups_per_unit(slices, h.ufi, h.ufk, wide);
        a.dealt = plan->d_items + (size_t)h.n_blocks * WAVES_PER_WG * ITEM_WORDS;
        a.n_dealt = dealt ? plan->n_dealt : 0;
        const uint64_t skipped = (uint64_t)j0 * 4u;
        a.b_bytes = wide || b_total <= skipped ? 0u : (uint32_t)(b_total - skipped);
        const int e = spmm_launch_chunks(a, h.ufi, h.ufk, slices, wide, plan->depth, stream);
        if (e != 0) return SPMM_ERR_HIP;
        j0 += cols;
    }
    return SPMM_OK;
}

}  // namespace

spmm_status_t spmm_execute(const spmm_plan_t *plan, const float *B, int32_t N, float *C, void *stream)
{
    return execute_with(plan, B, N, C, stream, plan ? plan->d_cross_sums : nullptr, CROSS_MAX_TILES);
}

spmm_status_t spmm_execute_static(const spmm_plan_t *plan, const float *B, int32_t N, float *C, void *stream)
{
    if (!plan) return SPMM_ERR_INVALID_ARG;
    const HostPlan &h = plan->host;
    if (h.k_slices > 1 && plan->on_device && plan->on_chunks()) return SPMM_ERR_UNSUPPORTED;  // the slices' buffer is beyond the static array
    if (h.n_cross_slots == 0 || !plan->on_device || !plan->on_chunks()) return execute_with(plan, B, N, C, stream, nullptr, 0);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return hip_fail();
    if (dev != plan->device) return SPMM_ERR_INVALID_ARG;
    float *sums = nullptr;
    size_t bytes = 0;
    if (spmm_static_scratch(&sums, &bytes) != 0) return hip_fail();
    // one column tile of a launch needs a slot of ufi x CROSS_ROW_FLOATS floats per workgroup of a cut panel
    const size_t per_tile = (size_t)h.n_cross_slots * (size_t)h.ufi * CROSS_ROW_FLOATS * sizeof(float);
    if (per_tile > bytes) return SPMM_ERR_UNSUPPORTED;
    const size_t tiles = bytes / per_tile;
    return execute_with(plan, B, N, C, stream, sums, (int32_t)(tiles < 65535 ? tiles : 65535));
}

spmm_status_t spmm_plan_destroy(spmm_plan_t *plan)
{
    if (!plan) return SPMM_OK;
    plan_release()(plan);
    return SPMM_OK;
}

spmm_status_t spmm_plan_describe_sized(const spmm_plan_t *plan, spmm_plan_info_t *out, size_t out_bytes)
{
    if (!plan || !out) return SPMM_ERR_INVALID_ARG;
    const HostPlan &h = plan->host;
    spmm_plan_info_t info;
    std::memset(&info, 0, sizeof info);
    info.M = h.M;
    info.K = h.K;
    info.nnz = h.nnz;
    info.ufi = h.ufi;
    info.ufk = h.ufk;
    info.group_nnz = h.group_nnz;
    info.group_panels = h.group_panels;
    info.n_groups = (int64_t)(h.groups.size() / 5);
    info.n_blocks = h.n_blocks;
    info.n_split = h.n_split;
    info.n_enum = h.n_enum;
    info.n_chunks = h.n_chunks;
    info.stream_words = plan->stream_words;
    info.device_bytes = plan->device_bytes;
    info.sorted_rows = h.rowmap.empty() ? 0 : 1;
    info.n_cross = h.n_cross;
    info.scratch_bytes = plan->scratch_bytes;
    info.k_slices = h.k_slices;
    info.slice_rows = h.slice_rows;
    info.slice_cols = h.slice_cols;
    info.tile_rows = plan->tiles.rows;
    info.strip_units = plan->strips.n_units;
    std::memset(out, 0, out_bytes);
    std::memcpy(out, &info, std::min(out_bytes, sizeof info));
    return SPMM_OK;
}

spmm_status_t(spmm_plan_describe)(const spmm_plan_t *plan, spmm_plan_info_t *out)
{
    return spmm_plan_describe_sized(plan, out, offsetof(spmm_plan_info_t, tile_rows));
}

spmm_status_t spmm_plan_get_groups(const spmm_plan_t *plan, int32_t *out, int64_t cap)
{
    if (!plan || !out) return SPMM_ERR_INVALID_ARG;
    const HostPlan &h = plan->host;
    const int64_t n = (int64_t)(h.groups.size() / 5);
    if (cap < n) return SPMM_ERR_INVALID_ARG;
    if (n) std::memcpy(out, h.groups.data(), (size_t)n * 5 * sizeof(int32_t));
    return SPMM_OK;
}

spmm_status_t spmm_plan_get_array(const spmm_plan_t *plan, int32_t which, uint32_t *out, int64_t cap_words,
                                  int64_t *n_words)
{
    if (!plan) return SPMM_ERR_INVALID_ARG;
    if (plan->on_device) return SPMM_ERR_INVALID_ARG;  // only host-only plans keep the mirror
    const HostPlan &h = plan->host;
    if (which == SPMM_ARRAY_ROWMAP) {
        // M entries for a plan with sorted rows (the vector carries padding for the kernel), else none
        const int64_t n = h.rowmap.empty() ? 0 : h.plan_rows;
        if (n_words) *n_words = n;
        if (!out) return SPMM_OK;
        if (cap_words < n) return SPMM_ERR_INVALID_ARG;
        if (n) std::memcpy(out, h.rowmap.data(), (size_t)n * 4);
        return SPMM_OK;
    }
    const uint32_t *words = nullptr;
    size_t count = 0;
    auto take = [&](const auto &v) {
        words = v.data();
        count = v.size();
    };
    switch (which) {
    case SPMM_ARRAY_HDR: take(h.hdr); break;
    case SPMM_ARRAY_STREAM: take(h.stream); break;
    case SPMM_ARRAY_WINS: take(h.wins); break;
    case SPMM_ARRAY_ITEMS: take(h.items); break;
    case SPMM_ARRAY_CROSS: take(h.cross); break;
    default: return SPMM_ERR_INVALID_ARG;
    }
    if (n_words) *n_words = (int64_t)count;
    if (!out) return SPMM_OK;
    if (cap_words < (int64_t)count) return SPMM_ERR_INVALID_ARG;
    if (count) std::memcpy(out, words, count * 4);
    return SPMM_OK;
}

// For the tests, which compare the strips of the two builders: the units, rows and groups of a plan on strips (as many words as
// fit `cap`); how many words they are, or -1.
int64_t spmm_strips_words(const spmm_plan_t *plan, uint32_t *out, int64_t cap, int32_t *built_on_device)
{
    if (!plan || !plan->on_device || plan->strips.n_units == 0) return -1;
    const StripPlan &p = plan->strips;
    const size_t front = (size_t)(p.n_units * (p.bands * 2 + 64)), behind = (size_t)(p.steps / STRIP_STEPS) * (STRIP_GROUP_BYTES / 4);
    if (built_on_device) *built_on_device = p.built_on_device;
    if (out && cap >= (int64_t)(front + behind) &&
        (hipMemcpy(out, p.d_units, front * 4, hipMemcpyDeviceToHost) != hipSuccess || hipMemcpy(out + front, p.d_stream, behind * 4, hipMemcpyDeviceToHost) != hipSuccess))
        return -1;
    return (int64_t)(front + behind);
}

// For the tests and the benchmark: the column tiles of the first launch on N columns of a plan on chunks, and the columns of one; 0
// on tiles and strips.
int32_t spmm_chunk_tiles(const spmm_plan_t *plan, int32_t N, int32_t *tile_cols)
{
    if (!plan || !plan->on_device || !plan->on_chunks() || N < 1) return 0;
    int32_t tile = 0, cols = 0;
    int slices = 0;
    const column_tiles tiling(*plan, N);
    const int32_t n = tiling.launch(tiling.sliced ? std::min(N, KSLICE_COLS) : N, tile, cols, slices);
    if (tile_cols) *tile_cols = tile;
    return n;
}

const char *spmm_status_string(spmm_status_t status)
{
    switch (status) {
    case SPMM_OK: return "ok";
    case SPMM_ERR_INVALID_ARG: return "invalid argument";
    case SPMM_ERR_INVALID_CSR: return "invalid CSR structure";
    case SPMM_ERR_ALLOC: return "allocation failed";
    case SPMM_ERR_HIP: return "HIP runtime error";
    case SPMM_ERR_UNSUPPORTED: return "size not supported";
    default: return "unknown status";
    }
}

}  // extern "C"
