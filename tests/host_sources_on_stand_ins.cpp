// The library's host sources on stand-ins: tests/test_host_sources.py compiles them together with this file, in
// which the HIP runtime and the kernels' entry points are stand-ins in host memory.
//   failures   every allocation of a plan's creation is made to fail in turn, also those on the device
//   choices    which matrices are left to chunks that strips would take by the lengths of their rows
//   launches   what spmm_execute hands to the launcher
//   places     what the workgroups of a launch compute
//   threads    how many threads a creation starts
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <pthread.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <thread>
#include <vector>

#include "spmm.h"
#include "spmm_kernels.h"
#include "spmm_strips.h"
#include "spmm_tiles.h"

// ---- host memory: allocation number `fail_at` fails, and everything is counted

static std::atomic<long> made{0}, fail_at{-1}, host_live{0};

void *operator new(size_t n)
{
    if (fail_at >= 0 && made++ == fail_at) throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    ++host_live;
    return p;
}
void operator delete(void *p) noexcept
{
    if (!p) return;
    --host_live;
    std::free(p);
}
void operator delete(void *p, size_t) noexcept { operator delete(p); }

// ---- threads: counted

static std::atomic<long> threads_started{0};

extern "C" int pthread_create(pthread_t *thread, const pthread_attr_t *attr, void *(*start)(void *), void *arg)
{
    typedef int (*function)(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *);
    static const function real = reinterpret_cast<function>(dlsym(RTLD_NEXT, "pthread_create"));
    ++threads_started;
    return real(thread, attr, start, arg);
}

// ---- device memory

static long device_live = 0, device_made = 0, device_fail_at = -1;
static bool memset_pending = false;  // hipMemset may return early; copies from the host do not

extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    if (device_made++ == device_fail_at) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    ++device_live;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    --device_live;
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind)
{
    std::memcpy(dst, src, n);
    memset_pending = false;
    return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n)
{
    std::memset(p, v, n);
    memset_pending = true;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

// ---- the device sources' entry points

static int tiles_status = 0;      // what the builder of tiles answers
static double tiles_time = 1e9;   // its estimate of a product's time

static std::vector<spmm_launch_args> launched;

int spmm_launch_chunks(const spmm_launch_args &a, int, int, int, bool, int, void *)
{
    launched.push_back(a);
    return 0;
}
int spmm_static_scratch(float **, size_t *) { return 1; }
int spmm_tiles_execute(const TilePlan &, int64_t, int64_t, const float *, int32_t, float *, void *) { return 0; }
double spmm_tiles_time(int, int64_t, int64_t, int64_t, double, double, int *) { return tiles_time; }
int spmm_tiles_build(int64_t, int64_t, const int32_t *, const int32_t *, const float *, int32_t rows, TilePlan &out)
{
    out = TilePlan();
    if (tiles_status != 0) return tiles_status;
    out.rows = rows;
    return hipMalloc(reinterpret_cast<void **>(&out.d_stream), 64) == hipSuccess ? 0 : 3;
}
void spmm_tiles_release(TilePlan &p)
{
    if (p.d_stream) (void)hipFree(p.d_stream);
    p = TilePlan();
}

static int strips_status = STRIPS_NOT_POSSIBLE;  // what the builder of strips on the device answers
static int strips_asked = 0;                     // how often

int spmm_strips_build_on_device(int64_t, int64_t, const int32_t *, const int32_t *, const float *, int64_t, strips::start &, StripPlan &out)
{
    out = StripPlan();
    ++strips_asked;
    if (strips_status != 0) return strips_status;
    out.n_units = 1;
    out.device_bytes = 64;
    return hipMalloc(reinterpret_cast<void **>(&out.d_units), 64) == hipSuccess ? 0 : 3;
}
int spmm_strips_execute(const StripPlan &, int64_t, const float *, int32_t, float *, void *) { return 0; }
void spmm_strips_release(StripPlan &p)
{
    if (p.d_units) (void)hipFree(p.d_units);
    p = StripPlan();
}

// ---- inputs

struct csr {
    int64_t M, K;
    std::vector<int32_t> row_ptr{0}, col_idx;
    std::vector<float> vals;
};

// Every `step`-th column of a row; the first `heavy` rows hold four times as many entries.
static csr matrix(int64_t M, int64_t K, int step, int heavy)
{
    csr a{M, K};
    for (int64_t i = 0; i < M; ++i) {
        const int s = i < heavy ? step / 4 : step;
        for (int64_t c = i % s; c < K; c += s) {
            a.col_idx.push_back((int32_t)c);
            a.vals.push_back((float)(c % 7) - 3.0f);
        }
        a.row_ptr.push_back((int32_t)a.col_idx.size());
    }
    return a;
}

static spmm_status_t create(const csr &a, const spmm_options_t &o, spmm_plan_t **p)
{
    return spmm_plan_create_ex(p, a.M, a.K, a.row_ptr.data(), a.col_idx.data(), a.vals.data(), &o);
}

#define REQUIRE(x) do { if (!(x)) { std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x); std::exit(1); } } while (0)

// Lets allocation after allocation fail, host and device, until a creation comes through: each failure has to
// be reported as one and leave nothing behind.
static void fail_in_turn(const char *name, const csr &a, const spmm_options_t &o)
{
    spmm_plan_t *p = nullptr;
    REQUIRE(create(a, o, &p) == SPMM_OK);
    REQUIRE(!memset_pending);  // any stream may execute the plan now
    REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
    for (int on_device = 0; on_device < 2; ++on_device) {
        long tried = 0, refused = 0;
        for (long n = 0;; ++n) {
            const long host_before = host_live, device_before = device_live;
            p = nullptr;
            made = 0;
            device_made = 0;
            fail_at = on_device ? -1 : n;
            device_fail_at = on_device ? n : -1;
            const spmm_status_t st = create(a, o, &p);
            fail_at = -1;
            device_fail_at = -1;
            const bool reached = on_device ? device_made > n : made > n;
            ++tried;
            REQUIRE(st == SPMM_OK || (st == SPMM_ERR_ALLOC && p == nullptr && reached));
            refused += st != SPMM_OK;
            REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
            REQUIRE(host_live == host_before && device_live == device_before);
            if (!reached) break;
        }
        std::printf("%s: %ld %s allocations made to fail, %ld creations refused\n", name, tried - 1, on_device ? "device" : "host", refused);
    }
}

static csr spread(int64_t K, double sigma, int64_t M = 1024, double mean = 0.1);

static void failures()
{
    spmm_options_t o;
    const csr dense = matrix(300, 1000, 2, 0);
    {   // the choice between chunks and tiles, one thread
        std::memset(&o, 0, sizeof o);
        o.threads = 1;
        fail_in_turn("chunks", dense, o);
        tiles_time = 0.0;
        spmm_plan_t *p = nullptr;
        spmm_plan_info_t info;
        REQUIRE(create(dense, o, &p) == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK && info.tile_rows > 0);
        REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
        fail_in_turn("tiles", dense, o);
        // executes share scratch memory on chunks, not on tiles: scratch_bytes tells
        const csr cut = matrix(512, 16384, 4, 0);
        for (int asked : {-1, 0}) {
            o.tiles = asked;
            REQUIRE(create(cut, o, &p) == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK && info.k_slices == 4);
            REQUIRE((info.tile_rows > 0) == (asked == 0) && (info.scratch_bytes > 0) == (asked < 0));
            REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
        }
        // no room for the tiles: chunks, also where tiles were asked for
        tiles_status = SPMM_ERR_ALLOC;
        for (int asked : {0, 16}) {
            o.tiles = asked;
            REQUIRE(create(dense, o, &p) == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK);
            REQUIRE(info.tile_rows == 0 && info.device_bytes > 0 && info.stream_words > 0);
            REQUIRE(spmm_plan_destroy(p) == SPMM_OK && device_live == 0);
        }
        for (int status : {SPMM_ERR_HIP, SPMM_ERR_INVALID_CSR}) {  // anything else is reported
            tiles_status = status;
            REQUIRE(create(dense, o, &p) == (spmm_status_t)status && p == nullptr && device_live == 0);
        }
        tiles_status = 0;
        tiles_time = 1e9;
    }
    {   // no room for the strips, on the device or on the host: chunks, also where strips were asked for
        std::memset(&o, 0, sizeof o);
        o.threads = 1;
        o.n_hint = 128;
        spmm_plan_t *p = nullptr;
        spmm_plan_info_t info;
        for (int asked : {0, 1}) {
            const csr a = spread(asked ? 400 : 4096, 0.0, asked ? 300 : 4096, 0.05);
            o.strips = asked;
            REQUIRE(create(a, o, &p) == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK && info.strip_units > 0);
            REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
            for (int status : {STRIPS_NOT_POSSIBLE, (int)SPMM_ERR_ALLOC}) {
                strips_status = status;
                device_made = 0;
                device_fail_at = 0;  // the first allocation is that of the strips
                const spmm_status_t st = create(a, o, &p);
                device_fail_at = -1;
                REQUIRE(st == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK);
                REQUIRE(info.strip_units == 0 && info.tile_rows == 0 && info.device_bytes > 0 && info.stream_words > 0);
                REQUIRE(spmm_plan_destroy(p) == SPMM_OK && device_live == 0);
            }
            for (int status : {SPMM_ERR_HIP, SPMM_ERR_INVALID_CSR}) {  // anything else is reported
                strips_status = status;
                REQUIRE(create(a, o, &p) == (spmm_status_t)status && p == nullptr && device_live == 0);
            }
            strips_status = STRIPS_NOT_POSSIBLE;
        }
        const csr a = spread(400, 0.0, 300, 0.05);
        fail_in_turn("strips", a, o);
        long on_chunks = 0;
        for (long n = 0; on_chunks == 0; ++n) {
            made = 0;
            fail_at = n;
            const spmm_status_t st = create(a, o, &p);
            fail_at = -1;
            REQUIRE(made > n);  // or no failure of the host's builder led to chunks
            if (st != SPMM_OK) continue;
            REQUIRE(spmm_plan_describe(p, &info) == SPMM_OK);
            on_chunks += info.strip_units == 0;
            REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
        }
    }
    {   // blocks dealt to the compute units (more than 512 of them)
        const csr uneven = matrix(1090, 2048, 16, 40);
        std::memset(&o, 0, sizeof o);
        o.threads = 1;
        o.n_hint = 64;
        o.ufi = 1;
        o.group_nnz = 32;
        spmm_plan_t *p = nullptr;
        spmm_plan_info_t info;
        REQUIRE(create(uneven, o, &p) == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK);
        std::printf("%lld workgroups\n", (long long)info.n_blocks);
        REQUIRE(info.n_blocks > 512 && info.n_blocks <= 640);
        REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
        fail_in_turn("dealt", uneven, o);
    }
    {   // several threads: their handles and their states are allocations too
        std::memset(&o, 0, sizeof o);
        o.threads = 4;
        fail_in_turn("four threads", dense, o);
        o.kslices = 4;
        o.sort_rows = 1;
        fail_in_turn("four threads, column ranges", matrix(300, 1000, 8, 20), o);
        o.kslices = 0;
        o.cross = 1;
        o.group_nnz = 16;
        fail_in_turn("four threads, panels across workgroups", matrix(300, 1000, 8, 20), o);
    }
}

// A matrix whose row lengths spread by `sigma` (lognormal).
static csr spread(int64_t K, double sigma, int64_t M, double mean)
{
    csr a{M, K};
    uint64_t state = 12345;
    auto uniform = [&] { return (double)((state = state * 6364136223846793005u + 1442695040888963407u) >> 11) / 9007199254740992.0; };
    for (int64_t i = 0; i < a.M; ++i) {
        double z = -6.0;
        for (int k = 0; k < 12; ++k) z += uniform();
        const double density = mean * std::exp(sigma * z - 0.5 * sigma * sigma);
        for (int64_t c = 0; c < K; ++c)
            if (uniform() < density) {
                a.col_idx.push_back((int32_t)c);
                a.vals.push_back(1.0f);
            }
        a.row_ptr.push_back((int32_t)a.col_idx.size());
    }
    return a;
}

static bool on_strips(const csr &a, int n_hint, int strips = 0)
{
    spmm_options_t o;
    std::memset(&o, 0, sizeof o);
    o.n_hint = n_hint;
    o.strips = strips;
    o.threads = 8;
    spmm_plan_t *p = nullptr;
    spmm_plan_info_t info;
    REQUIRE(create(a, o, &p) == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK && info.tile_rows == 0);
    REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
    return info.strip_units > 0;
}

// The matrix with its column c as column c * by + i % turn of row i.
static csr stretched(csr a, int by, int turn = 1)
{
    a.K *= by;
    for (int64_t i = 0; i < a.M; ++i)
        for (int32_t q = a.row_ptr[(size_t)i]; q < a.row_ptr[(size_t)i + 1]; ++q) a.col_idx[(size_t)q] = a.col_idx[(size_t)q] * by + (int32_t)(i % turn);
    return a;
}

// The builder on the device refuses everything here (STRIPS_NOT_POSSIBLE), so the host's makes the strips.
static void choices()
{
    const csr even = spread(4096, 0.0, 4096, 0.05);
    REQUIRE(on_strips(even, 128));
    // columns of which many are the same modulo 8 collide in LDS
    for (int by : {2, 4, 8}) {
        const csr a = stretched(spread(4096 / by, 0.0, 4096, 0.05 * by), by);
        REQUIRE(on_strips(a, 128) == (by == 2) && on_strips(a, 128, 1));
    }
    REQUIRE(!on_strips(stretched(spread(512, 0.0, 4096, 0.4), 8, 8), 128));
    // ... but where chunks take twice as long as strips those may take half as long again
    REQUIRE(on_strips(stretched(spread(628, 0.3, 3001, 0.6), 4), 200));
    // without a hint in bands: slower than chunks at one of the widths that those have tuned kernels for
    REQUIRE(!on_strips(spread(13276, 0.0, 3071, 0.093), 0) && on_strips(spread(13276, 0.0, 3071, 0.093), 200) && on_strips(spread(2511, 0.5, 3001, 0.15), 0));
    // ... which the estimates tell of rows that are not skewed only
    REQUIRE(on_strips(spread(8330, 2.0, 2167, 0.05), 0));
    // short rows, eight entries on average, are looked at together
    REQUIRE(on_strips(spread(512, 0.0, 32768, 0.016), 200) && !on_strips(stretched(spread(64, 0.0, 32768, 0.125), 8), 200));
}

// spmm_execute's launches of a chunk plan of `a`, made for 64 columns, on N columns.
static std::vector<spmm_launch_args> launches(const csr &a, int N, spmm_plan_info_t *info)
{
    static float word;  // B and C are only passed on
    spmm_options_t o;
    std::memset(&o, 0, sizeof o);
    o.n_hint = 64;
    o.tiles = -1;
    spmm_plan_t *p = nullptr;
    REQUIRE(create(a, o, &p) == SPMM_OK && spmm_plan_describe(p, info) == SPMM_OK);
    launched.clear();
    REQUIRE(spmm_execute(p, &word, N, &word, nullptr) == SPMM_OK);
    REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
    return launched;
}

// A few more than 512 workgroups of uneven rows, which would overload the units that get three, are dealt by weight; not even
// rows, and not where several column tiles share the launch.  Compute units are held to two workgroups (extra LDS) for tiles
// of 64 columns that fill an L2 only.
static void dealt_or_held()
{
    spmm_plan_info_t info;
    for (int N : {64, 100, 128}) {
        const std::vector<spmm_launch_args> uneven = launches(spread(4096, 0.5), N, &info);
        REQUIRE(info.ufi == 1 && info.n_blocks > 512 && info.n_blocks <= 640);
        REQUIRE(uneven.size() == 1 && uneven[0].n_tiles == 1 && uneven[0].n_dealt > 512 && uneven[0].lds_pad == 0);
    }
    const std::vector<spmm_launch_args> two_tiles = launches(spread(4096, 0.5), 256, &info);
    REQUIRE(two_tiles.size() == 1 && two_tiles[0].n_tiles == 2 && two_tiles[0].n_dealt == 0 && two_tiles[0].lds_pad == 0);
    const std::vector<spmm_launch_args> even = launches(matrix(1024, 4096, 10, 0), 64, &info);
    REQUIRE(even[0].n_dealt == 0 && even[0].lds_pad == 0);
    const std::vector<spmm_launch_args> filled = launches(spread(16384, 0.0, 300, 0.02), 128, &info);
    REQUIRE(filled.size() == 1 && filled[0].n_tiles == 2 && filled[0].tile_cols == 64 && filled[0].lds_pad == 24u << 10);
}

// Every block of every tile exactly once: the first `front` blocks of all tiles, block by block, then the others tile by tile.
static void places_of(uint32_t n_blocks, uint32_t n_tiles, uint32_t front)
{
    uint32_t block = 0, tile = 0;  // expected
    for (uint32_t y = 0; y < n_tiles; ++y)
        for (uint32_t x = 0; x < n_blocks; ++x) {
            const place p = place_of(launch_shape{n_blocks, n_tiles, front}, launch_group{x, y});
            REQUIRE(p.block == block && p.tile == tile);
            if (block < front) {
                if (++tile == n_tiles) {
                    tile = 0;
                    ++block;
                }
            } else if (++block == n_blocks) {
                block = front;
                ++tile;
            }
        }
    REQUIRE(front == n_blocks ? block == n_blocks : tile == n_tiles);
}

static void places()
{
    for (uint32_t n_blocks = 1; n_blocks <= 70; ++n_blocks)
        for (uint32_t n_tiles = 1; n_tiles <= 20; ++n_tiles)
            for (uint32_t front = 0; front <= n_blocks; ++front) places_of(n_blocks, n_tiles, front);
    for (uint32_t front : {0u, 1u, 128u, 256u, 4999u, 5000u}) places_of(5000, 5, front);
    // the largest launches: workgroups of 256 threads, fewer than 2^32 of these in a row of the grid
    const uint32_t most = (1u << 24) - 1;
    const launch_shape wide{most, 256, 1}, whole_front{most, 8, most};
    const place first = place_of(wide, launch_group{0, 0}), last = place_of(wide, launch_group{most - 1, 255}), end = place_of(whole_front, launch_group{most - 1, 7});
    REQUIRE(first.block == 0 && first.tile == 0 && last.block == most - 1 && last.tile == 255 && end.block == most - 1 && end.tile == 7);
    // the rule's choices, at the edges of its widths, for plans of few and many, even and uneven blocks
    uint32_t whole = 0, some = 0, none = 0;
    for (int64_t M : {300, 1024, 3000})
        for (double sigma : {0.0, 0.7}) {
            const csr a = spread(700, sigma, M);
            for (int N : {64, 128, 129, 160, 161, 176, 192, 200, 239, 240, 256, 300, 384, 495, 496, 512, 1008, 1024, 1100, 40000}) {
                spmm_plan_info_t info;
                for (const spmm_launch_args &l : launches(a, N, &info)) {
                    const uint32_t front = front_blocks(l), n = (uint32_t)l.n_blocks;
                    REQUIRE(front <= n && (front < n || l.n_tiles <= 256));
                    places_of(n, (uint32_t)l.n_tiles, front);
                    (front == 0 ? none : front == n ? whole : some) += 1;
                }
            }
        }
    std::printf("launches: %u tile by tile, %u some blocks first, %u block by block\n", none, some, whole);
    REQUIRE(none > 0 && some > 0 && whole > 0);
}

// Plans of single rows with fewer than 2^20 entries are made by one thread where the columns ascend, and by several where many
// rows have to be sorted first; the plans are the same.
static void threads()
{
    csr ordered = spread(4096, 0.0, 1024, 0.1);
    for (size_t q = 0; q < ordered.vals.size(); ++q) ordered.vals[q] = (float)q;
    REQUIRE(ordered.vals.size() > (size_t)1 << 18 && ordered.vals.size() < (size_t)1 << 20);
    if (std::thread::hardware_concurrency() < 2) return;
    std::vector<uint32_t> arrays[3];
    long started[3];
    for (int k = 0; k < 3; ++k) {  // rows turned around: none, the first ten, all
        csr a = ordered;
        for (int64_t i = 0; i < (k == 0 ? 0 : k == 1 ? 10 : a.M); ++i) {
            std::reverse(a.col_idx.begin() + a.row_ptr[(size_t)i], a.col_idx.begin() + a.row_ptr[(size_t)i + 1]);
            std::reverse(a.vals.begin() + a.row_ptr[(size_t)i], a.vals.begin() + a.row_ptr[(size_t)i + 1]);
        }
        spmm_options_t o;
        std::memset(&o, 0, sizeof o);
        o.host_only = 1;
        o.n_hint = 64;
        spmm_plan_t *p = nullptr;
        spmm_plan_info_t info;
        const long before = threads_started;
        REQUIRE(create(a, o, &p) == SPMM_OK && spmm_plan_describe(p, &info) == SPMM_OK && info.ufi == 1);
        started[k] = threads_started - before;
        for (int which : {SPMM_ARRAY_HDR, SPMM_ARRAY_STREAM, SPMM_ARRAY_WINS, SPMM_ARRAY_ITEMS}) {
            int64_t n = 0;
            REQUIRE(spmm_plan_get_array(p, which, nullptr, 0, &n) == SPMM_OK);
            const size_t at = arrays[k].size();
            arrays[k].resize(at + (size_t)n);
            REQUIRE(spmm_plan_get_array(p, which, arrays[k].data() + at, n, nullptr) == SPMM_OK);
        }
        REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
    }
    std::printf("threads started: %ld, %ld and %ld\n", started[0], started[1], started[2]);
    REQUIRE(started[0] == 0 && started[1] == 0 && started[2] > 0);
    REQUIRE(arrays[0] == arrays[1] && arrays[0] == arrays[2]);
}

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "failures")) failures();
    else if (!std::strcmp(what, "choices")) choices();
    else if (!std::strcmp(what, "launches")) dealt_or_held();
    else if (!std::strcmp(what, "places")) places();
    else if (!std::strcmp(what, "threads")) threads();
    else return 2;
    std::printf("ok\n");
    return 0;
}
