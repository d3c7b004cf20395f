// gfx950 executor and builder of the matrix-core path: C <- A x B with A in tiles
// (format: spmm_tiles.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "spmm_launch.h"
#include "spmm_places.h"
#include "spmm_tiles.h"
#include "spmm_upload.h"

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_unaligned __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int OPS = TILE_OPERANDS;
constexpr int NARROW_ROWS = 8;
constexpr int A_SLOT_WORDS = TILE_PLACE0 / 4 + 1024;  // the expanded block behind the dump word

// ---------------------------------------------------------------- executor

struct tile_args {
    const uint32_t *stream, *offsets;
    const float *B;
    float *C;
    uint64_t b_bytes;   // bytes of B
    int32_t n_panels, n_steps, n_tiles, M, K, N;
    uint32_t first;     // the launch's first place among all column tiles of all panels
    float largest;      // size of A's largest value (spmm_split_tiles_kernel)
    uint32_t set;       // column tiles that come first, of all panels (panels of 16 rows; tiles_of_set)
};

template <int NB> struct BVec;
template <> struct BVec<1> { typedef float type; };
template <> struct BVec<2> { typedef f32x2 type; };
template <> struct BVec<4> { typedef f32x4 type; };

__device__ __forceinline__ float part(float v, int) { return v; }
__device__ __forceinline__ float part(const f32x2 &v, int j) { return v[j]; }
__device__ __forceinline__ float part(const f32x4 &v, int j) { return v[j]; }

template <int NB> __device__ __forceinline__ typename BVec<NB>::type buffer_load(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    if constexpr (NB == 1) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
    else if constexpr (NB == 2) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
        return f32x2{__uint_as_float(v[0]), __uint_as_float(v[1])};
    } else {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
        return f32x4{__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3])};
    }
}

// What the lanes of a wave wrote to LDS before this point is what they read after it.
__device__ __forceinline__ void lds_in_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int R> struct Tile;
template <> struct Tile<32> {
    typedef f32x16 acc_t;
    static constexpr int GROUPS = 4;  // groups of four accumulator registers
    static __device__ __forceinline__ acc_t mfma(float b, float a, const acc_t &c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(b, a, c, 0, 0, 0); }
    static __device__ __forceinline__ acc_t mfma(const bf16x8 &b, const bf16x8 &a, const acc_t &c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(b, a, c, 0, 0, 0); }
};
template <> struct Tile<16> {
    typedef f32x4 acc_t;
    static constexpr int GROUPS = 1;
    static __device__ __forceinline__ acc_t mfma(float b, float a, const acc_t &c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(b, a, c, 0, 0, 0); }
};

// The workgroup's place among the column tiles of all panels, panel by panel.  Workgroups are dealt to
// the eight XCDs in turn: each XCD takes an eighth of these places, next to each other, so that a panel's
// blocks are read into one L2 (but for the panels at the borders) and the XCDs have equally much to do
// also when the panels are few (269 x 6139, 82 % pruned, 100 columns: with whole panels dealt to XCDs 16.5 us, now 12.5).
__device__ __forceinline__ uint32_t place_in_matrix(uint32_t first) { return first + blockIdx.x % 8u * (gridDim.x / 8u) + blockIdx.x / 8u; }

// Of the waves of a SIMD the one that started first would go first, and the workgroup waits for the last: at the end of equally many
// steps 3.3, 4.2, 4.5 and 5.1 us (512 x 2048, 80 % pruned, 128 columns), and matrix and vector instructions of fewer and fewer waves beside each other
// before it.  The wave with more steps left goes first, in four classes that get narrower towards the end.  Steps left of as many as the
// workgroup's busiest wave has: of a wave's own, one with its only step to come would be as urgent as one with two (8137 x 328, 66 %, 102 columns 9.4 -> 9.7 us).
//   512 x 2048, 80 %, 128 columns       6.4 -> 6.1 us     8192 x 2048, 50 %, 64 columns     19.9 -> 19.1 us
//   4096 x 1024, 70 %, 128 columns     11.3 -> 10.9       7872 x 2688, 87 %, 140 columns    58.6 -> 55.9
//   4096 x 4096, 50 %, 128 columns     33.7 -> 32.3       8192 x 8192, 50 %, 128 columns   108.0 -> 105.5
// Thirty products 2.5 % on average, none of them 1 % slower; classes at equal distances 2 %.  (Panels of 8 rows: between 2 % faster and 3 % slower, not there.)
__device__ __forceinline__ void first_if_behind(uint32_t left, uint32_t all)
{
    if (left * 2u > all) __builtin_amdgcn_s_setprio(3);
    else if (left * 4u > all) __builtin_amdgcn_s_setprio(2);
    else if (left * 8u > all) __builtin_amdgcn_s_setprio(1);
    else __builtin_amdgcn_s_setprio(0);
}

// Launches `kernel` for all column tiles of all panels.  HIP refuses a grid of 2^32 threads or more, which
// a C of 8 GiB reaches on panels of 8 rows (32768 x 65536): the places are dealt to as many launches as
// that takes.  (A C that fits the device's memory has fewer than 2^32 places.)
template <typename F> hipError_t launch_places(F kernel, tile_args &a, unsigned threads, hipStream_t s)
{
    const int64_t places = (int64_t)a.n_panels * a.n_tiles, most = (((int64_t)1 << 32) - 1) / threads / 8 * 8;
    for (int64_t first = 0; first < places; first += most) {
        a.first = (uint32_t)first;
        const unsigned blocks = (unsigned)((std::min(places - first, most) + 7) / 8) * 8u;
        const hipError_t e = launch_kernel(kernel, dim3(blocks), threads, 0, s, a);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The sum of the waves' tiles, in a fixed order: the upper half of the waves parks its tiles in LDS, the lower half adds
// them to its own, then all waves share the rest of the sum (store_sum).  `meanwhile` is called when all waves are there.
template <int R, int NB, int W, typename F> __device__ __forceinline__ void add_halves(const typename Tile<R>::acc_t (&acc)[NB], float *lds, int wave, int lane,
                                                                                      F meanwhile)
{
    constexpr int QUADS = NB * Tile<R>::GROUPS;
    f32x4 quad[QUADS];
#pragma unroll
    for (int f = 0; f < QUADS; ++f) {
        const int g = f / NB, q = f % NB;
#pragma unroll
        for (int x = 0; x < 4; ++x) quad[f][x] = acc[(4 * q + x) % NB][4 * g + (4 * q + x) / NB];
    }
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);
    __syncthreads();
    if (wave >= W / 2) {
#pragma unroll
        for (int f = 0; f < QUADS; ++f) red[((wave - W / 2) * QUADS + f) * 64 + lane] = quad[f];
    }
    meanwhile();
    __syncthreads();
    if (wave < W / 2) {
#pragma unroll
        for (int f = 0; f < QUADS; ++f) {
            f32x4 *p = &red[(wave * QUADS + f) * 64 + lane];
            *p = quad[f] + *p;
        }
    }
    __syncthreads();
}
// Calls `stored` with the first of every four columns and their sums.
template <int R, int NB, int W, typename F> __device__ __forceinline__ void store_sum(const tile_args &args, const float *lds, uint32_t panel, uint32_t n0, int wave,
                                                                                     int lane, F stored)
{
    constexpr int KO = 64 / R, QUADS = NB * Tile<R>::GROUPS;
    const f32x4 *red = reinterpret_cast<const f32x4 *>(lds);
    const uint32_t N = (uint32_t)args.N, row = panel * (uint32_t)R + (uint32_t)(lane % R);
    if (row >= (uint32_t)args.M) return;
#pragma unroll
    for (int f0 = 0; f0 < QUADS; f0 += W) {
        const int f = f0 + wave;
        if (f >= QUADS) break;
        f32x4 sum = red[f * 64 + lane];
#pragma unroll
        for (int u = 1; u < W / 2; ++u) sum += red[(u * QUADS + f) * 64 + lane];
        const uint32_t n = n0 + (uint32_t)(NB * (4 * KO * (f / NB) + 4 * (lane / R)) + 4 * (f % NB));
        float *dst = args.C + (size_t)row * N + n;
        if (n + 4 <= N) {
            *reinterpret_cast<f32x4_unaligned *>(dst) = sum;
        } else {
            for (uint32_t x = 0; x < 4; ++x)
                if (n + x < N) dst[x] = sum[(int)x];
        }
        stored(n, sum);
    }
}

// One workgroup computes a tile of C: R rows x NB * R columns.
//
// R       rows of a panel (32: v_mfma_f32_32x32x2, 16: v_mfma_f32_16x16x4; fp32 operands and sums)
// NB      column groups of the tile.  Lane l holds columns NB * (l % R) .. + NB - 1 of a row of B, so
//         that one load of NB words feeds NB matrix instructions
// W       waves of the workgroup; they share the tile and cut K: wave w multiplies steps w, w + W, ...
//         of the panel, which keeps the workgroup's rows of B together in the L2, and the waves'
//         partial tiles meet in LDS at the end, in a fixed order
// STAGED  rows of B pass through LDS (loads of one word per lane would cost the address path as much
//         as loads of four: 16 cycles each); wider tiles load them straight into registers
// WIDE    64-bit addresses of B, word by word: for the few N whose rows of a step span 4 GiB
//
// A wave's step: its block's entries, fetched one step ahead (16-byte loads), are scattered to their
// places in a zeroed 4 KiB slot of LDS, read back as 16 operands per lane (four 16-byte reads), the
// slot is zeroed again for the next block, and 16 * NB matrix instructions multiply.
//
// (32 rows x 128 and 64 columns: WIDE, values of A without exact parts, few steps; spmm_split_tiles_kernel below has the others.)
//
// What bounds it: the matrix cores' fp32 rate (157 TFLOP/s dense, 156 measured) times the density.  fp32
// matrix instructions issue from the vector ALUs (baselines/microbench_paths.hip: a 32x32x2 takes 64.6 cycles, 16
// integer adds 44.5, both together 108.7), so every vector instruction beside them costs: expanding the
// blocks from bitmaps in registers took 48 to 130 vector instructions per step, with the scatter a step has 30
// in all beside its matrix instructions, for 6 bytes per entry instead of 4.3.
template <int R, int NB, int W, bool STAGED, bool WIDE, int MINW>
__global__ __launch_bounds__(64 * W, MINW) void spmm_tiles_kernel(const tile_args args)
{
    typedef typename BVec<NB>::type bvec_t;
    typedef typename Tile<R>::acc_t acc_t;
    constexpr int KO = 64 / R;        // columns of A per operand
    constexpr int KS = OPS * KO;      // ... per step
    constexpr int NT = NB * R;        // columns of C per tile
    constexpr int QUADS = NB * Tile<R>::GROUPS;
    constexpr int B_SLOT_FLOATS = STAGED ? KS * NT : 0;
    constexpr int B_LOADS = STAGED ? KS * NT / 256 : 1;
    constexpr int SLOT = A_SLOT_WORDS + B_SLOT_FLOATS;
    constexpr int RED = (W / 2) * QUADS * 256;
    constexpr int LDS_WORDS = W * SLOT > RED ? W * SLOT : RED;
    __shared__ __attribute__((aligned(16))) float lds[LDS_WORDS];

    const uint32_t id = place_in_matrix(args.first);
    const set_place at = R == 16 ? place_in_sets(id, (uint32_t)args.n_panels, (uint32_t)args.n_tiles, args.set)
                                 : set_place{id / (uint32_t)args.n_tiles, id % (uint32_t)args.n_tiles};
    const uint32_t panel = at.row, nt = at.column;
    if (panel >= (uint32_t)args.n_panels) return;
    const uint32_t n0 = nt * (uint32_t)NT;

    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    float *slot = lds + wave * SLOT;
    float *bslot = slot + A_SLOT_WORDS;
    const uint32_t n_steps = (uint32_t)args.n_steps;
    const uint32_t *off_p = args.offsets + (size_t)panel * (n_steps + 1);
    const uint32_t N = (uint32_t)args.N;
    const uint32_t count = n_steps > (uint32_t)wave ? (n_steps - (uint32_t)wave + W - 1) / W : 0u;  // steps of this wave
    const uint32_t most = (n_steps + W - 1) / W;                                                                    // of any

    acc_t acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = acc_t{};

    // descriptor of the rows of B from step s on
    auto b_rsrc = [&](uint32_t s) {
        const uint64_t skip = ((uint64_t)s * KS * N + n0) * 4u;
        const uint64_t left = args.b_bytes > skip ? args.b_bytes - skip : 0u;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(args.B)) + skip, (short)0,
                                                 (int)(left > 0xFFFFFFFCull ? 0xFFFFFFFCu : (uint32_t)left), 0x00020000);
    };
    const uint32_t lane_off = ((uint32_t)(lane / R) * N + (uint32_t)(NB * (lane % R))) * 4u;                       // direct loads
    const uint32_t stage_off = ((uint32_t)(lane * 4 / NT) * N + (uint32_t)(lane * 4 % NT)) * 4u;                   // staged loads
    const uint32_t op_pitch = (uint32_t)KO * N * 4u, stage_pitch = (uint32_t)(256 / NT) * N * 4u;

    {
        f32x4 *z = reinterpret_cast<f32x4 *>(slot + TILE_PLACE0 / 4) + lane;
#pragma unroll
        for (int q = 0; q < OPS / 4; ++q) z[64 * q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    uint32_t lo = 0, hi = 0;  // lane i: bounds of the block of step 64 * (batch) + i of this wave
    f32x4 va[4];   // values of the block in flight, 256 entries at a time
    u32x2 vp[4];   // their places in the expanded block
    uint32_t n_next = 0;
    auto fetch_a = [&](uint32_t i) {
        if ((i & 63u) == 0) {
            const uint32_t s = (uint32_t)wave + W * (i + (uint32_t)lane);
            lo = s < n_steps ? off_p[s] : 0u;
            hi = s < n_steps ? off_p[s + 1] : 0u;
        }
        const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)(i & 63u));
        n_next = 8u * ((uint32_t)__builtin_amdgcn_readlane((int)hi, (int)(i & 63u)) - a);
        const char *block = reinterpret_cast<const char *>(args.stream) + (size_t)a * 48u;
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(block), (short)0, (int)(n_next * 4u), 0x00020000);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(block) + (size_t)n_next * 4u, (short)0, (int)(n_next * 2u), 0x00020000);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q == 0 || n_next > 256u * (uint32_t)q) {
                va[q] = buffer_load<4>(rv, (uint32_t)lane * 16u + 1024u * (uint32_t)q);
                vp[q] = __builtin_amdgcn_raw_buffer_load_b64(rp, (int)((uint32_t)lane * 8u + 512u * (uint32_t)q), 0, 0);
            }
    };
    f32x4 vb[B_LOADS];
    auto fetch_b = [&](uint32_t i) {
        const __amdgpu_buffer_rsrc_t r = b_rsrc((uint32_t)wave + W * i);
#pragma unroll
        for (int q = 0; q < B_LOADS; ++q) vb[q] = buffer_load<4>(r, stage_off + (uint32_t)q * stage_pitch);
    };
    constexpr int BATCH = NB == 2 && W == 16 ? 4 : 8;  // operands whose rows of B are requested together
    bvec_t bq[2][BATCH];
    auto fetch_batch = [&](__amdgpu_buffer_rsrc_t r, int k) {
#pragma unroll
        for (int t = 0; t < BATCH; ++t) bq[k % 2][t] = buffer_load<NB>(r, lane_off + (uint32_t)(k * BATCH + t) * op_pitch);
    };
    auto fetch_batch_wide = [&](uint32_t s, int k) {  // rows and columns outside B repeat its last ones (never used)
#pragma unroll
        for (int t = 0; t < BATCH; ++t) {
            const uint64_t row = (uint64_t)s * KS + (uint32_t)((k * BATCH + t) * KO + lane / R);
            const float *p = args.B + (row < (uint64_t)args.K ? row : (uint64_t)args.K - 1u) * N;
            if constexpr (NB == 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t n = n0 + (uint32_t)(4 * (lane % R) + j);
                    bq[k % 2][t][j] = p[n < N ? n : N - 1u];
                }
        }
    };
    auto fetch_rows = [&](uint32_t s, int k) {
        if constexpr (WIDE) fetch_batch_wide(s, k);
        else fetch_batch(b_rsrc(s), k);
    };

    if (count > 0) {
        fetch_a(0);
        if constexpr (STAGED) fetch_b(0);
        else fetch_rows((uint32_t)wave, 0);
        for (uint32_t i = 0; i < count; ++i) {
            first_if_behind(count - i, most);
            // ---- this step's entries (and rows of B) go to the wave's slot: every entry to its
            //      place in the expanded block, which is all zeros at this point
            const uint32_t n = n_next;
            char *cslot = reinterpret_cast<char *>(slot);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q == 0 || n > 256u * (uint32_t)q) {
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        *reinterpret_cast<float *>(cslot + ((vp[q][x / 2] >> (16 * (x % 2))) & 0xFFFFu)) = va[q][x];
                }
            if constexpr (STAGED) {
#pragma unroll
                for (int q = 0; q < B_LOADS; ++q) reinterpret_cast<f32x4 *>(bslot)[lane + 64 * q] = vb[q];
            }
            lds_in_order();
            // ---- the next step's data
            const bool more = i + 1 < count;
            if (more) {
                fetch_a(i + 1);
                if constexpr (STAGED) fetch_b(i + 1);
            }
            // ---- the lane's 16 values of A, and zeros for the next block
            f32x4 *z = reinterpret_cast<f32x4 *>(slot + TILE_PLACE0 / 4) + lane;
            f32x4 a4[OPS / 4];
#pragma unroll
            for (int q = 0; q < OPS / 4; ++q) a4[q] = z[64 * q];
#pragma unroll
            for (int q = 0; q < OPS / 4; ++q) z[64 * q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            // ---- multiply
            auto multiply = [&](int t, const bvec_t &bt) {
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[j] = Tile<R>::mfma(part(bt, j), a4[t / 4][t % 4], acc[j]);
            };
            if constexpr (STAGED) {
#pragma unroll
                for (int t = 0; t < OPS; ++t) multiply(t, *reinterpret_cast<const bvec_t *>(bslot + (t * 64 + lane) * NB));
            } else {
#pragma unroll
                for (int k = 0; k < OPS / BATCH; ++k) {
                    if (k + 1 < OPS / BATCH) fetch_rows((uint32_t)wave + W * i, k + 1);
                    else if (more) fetch_rows((uint32_t)wave + W * (i + 1), 0);
#pragma unroll
                    for (int t = 0; t < BATCH; ++t) multiply(k * BATCH + t, bq[k % 2][t]);
                }
            }
        }
    }

    add_halves<R, NB, W>(acc, lds, wave, lane, [] {});
    store_sum<R, NB, W>(args, lds, panel, n0, wave, lane, [](uint32_t, const f32x4 &) {});
}

// Column tiles of the first of two sets, whole lines of B, or all.  In one set every XCD fetches all of B into its L2 before its
// workgroups multiply, and an eighth of the blocks; in two, one set's places before the other's, half of B and a quarter of the blocks.  That
// pays where the blocks are few beside B and rows are whole lines.  Panels of 16 rows, plans and B in turn, in one set and in two, us:
//   entries / B   0.6   256 x 2048, 70 %, 192 columns  7.06 and 6.73     300 x 6000, 80 % lognormal, 160  13.4 and 12.9
//                 0.9   512 x 2048, 70 %, 256          9.48 and 9.23     512 x 4096, 85 %, 128            10.1 and 10.0
//                 1.2   512 x 2048, 80 %, 128          6.68 and 5.99
//                 3.8   1024 x 2048, 70 %, 128         9.12 and 9.11     (32 rows: 4096 x 1024, 70 %, 128, 15: 12.2 and 12.4)
// Rows that are not whole lines: 512 x 2048, 75 %, 100 columns 6.69 and 7.00.
// 11 random products that it takes 2.5 % faster on average, 1 % slower at worst; 49 others 0.93 to 1.06 times as fast in two sets, 0.99 on average.
uint32_t tiles_of_set(int tile_cols, uint32_t tiles, int64_t K, int32_t N, int64_t stream_words)
{
    const uint32_t line = tile_cols < 32 ? 32 / (uint32_t)tile_cols : 1, half = ((tiles + 1) / 2 + line - 1) / line * line;
    return N % 32 == 0 && 4.0 * (double)stream_words < 1.5 * 4.0 * (double)K * (double)N && half < tiles ? half : tiles;
}

template <int R, int NB, int W, bool STAGED, int MINW, bool WIDE = false> hipError_t launch(tile_args &a, hipStream_t s, int64_t stream_words = INT64_MAX)
{
    a.n_tiles = (int32_t)(((int64_t)a.N + NB * R - 1) / (NB * R));
    a.set = tiles_of_set(NB * R, (uint32_t)a.n_tiles, a.K, a.N, stream_words);
    return launch_places(spmm_tiles_kernel<R, NB, W, STAGED, WIDE, MINW>, a, 64 * W, s);
}

// ---------------------------------------------------------------- executor, fp32 values in three bf16 parts

// Eight values as h + m + l: the value rounded to bf16, what is left rounded to bf16, and what is left of that.  A
// float has 24 significant bits, a part 8 and a sign, and a value between 1 and 2 leaves at most 2^-8 and then 2^-17, a
// multiple of 2^-23: the sum is exact.  Only where the last part falls below the smallest bf16 (values under
// 2^-110) is it not: less than 2^-133 is lost, and `lost`, if asked for, gets a bit among its lower 16.  A value of
// 2^128 - 2^119 and more has an infinite h.
struct parts {
    bf16x8 h, m, l;
};
template <bool LOST> __device__ __forceinline__ parts in_parts(const float (&x)[8], uint32_t &lost)
{
    u32x4 h, m, l;
    float r[8];
    auto rounded = [](float lower, float upper) {  // (a conversion of a vector would be done twice, once for each way its result is used)
        uint32_t two;
        asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(two) : "v"(lower), "v"(upper));
        return two;
    };
    auto value = [](const u32x4 &p, int i) { return __uint_as_float(i % 2 ? p[i / 2] & 0xFFFF0000u : p[i / 2] << 16); };
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = rounded(x[2 * i], x[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = x[i] - value(h, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) m[i] = rounded(r[2 * i], r[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] -= value(m, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        l[i] = __builtin_amdgcn_perm(__float_as_uint(r[2 * i + 1]), __float_as_uint(r[2 * i]), 0x07060302u);
        if (LOST) lost |= __float_as_uint(r[2 * i]) | __float_as_uint(r[2 * i + 1]);
    }
    return parts{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
// What the parts are made of is not used after this point.  (The compiler would keep all terms of `lost` until the end.)
__device__ __forceinline__ void parts_done(parts &p, uint32_t &lost) { asm volatile("" : "+v"(p.h), "+v"(p.m), "+v"(p.l), "+v"(lost)); }

// N KiB from the start of `r` to `to`.  The load's last offset, a constant of the instruction, counts in both memories.
template <int N> __device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, float *to, int lane)
{
    if constexpr (N > 1) load_to_lds<N - 1>(r, to, lane);
    constexpr int Q = N - 1;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(to + 1024 * (Q / 4)), 16, lane * 16 + 4096 * (Q / 4), 0,
                                             1024 * (Q % 4), 0);
}

// Tiles of 32 rows x 128 or 64 columns on the bf16 matrix instructions (v_mfma_f32_32x32x16, sixteen times the
// products per cycle of the fp32 ones): every fp32 product is the sum of six products of parts,
// h h + (h m + m h) + (m m + h l + l h), which the instructions multiply exactly and add in fp32.  The three that are left
// out are below 2^-24 of the product, 2^-28 on average.  The sums of h h and of the five small ones are kept apart and added at the end: the large
// sums are then rounded once per 16 columns of A, where the fp32 instructions round once per two.  Error of the result (2-norm,
// against 64 bits) and that of fp32 instructions in tiles of 16 rows: 8192 x 8192, 50 % pruned, 128 columns 1.5e-7 and 4.1e-7; 4096 x 600 with 64, 8, 2 and
// 1 entries in every row 6.3e-8 and 7.6e-8, 5.32e-8 and 5.33e-8, 3.63e-8 and 3.62e-8, 2.59e-8 and 2.52e-8.
//
// Where sums are not finite the workgroup multiplies again, with fp32 instructions, and gives what the kernel above gives.  Plans with values of A that have no exact parts run on that kernel (TilePlan::exact_parts).  Where values of B have
// none, an element of C is off by at most 2^-133 x the largest value of A x K.  To an element 2^32 times as large that is
// nothing; where one is smaller, of a row with entries and a column near such a value, the workgroup multiplies again too.
// (8192 x 8192, 50 % pruned, 128 columns, 111 us: 111 with a tenth of B below 2^-110, 240 with a column of such values only or with
// an infinite one, 134 with such a value in A; 4096 x 1024, 70 % pruned, in tiles of 64, 11.0 us: 11.2, 22 and 12.2.)
//
// RUNS    runs of 256 entries that hold any block of the plan
// NB      column groups of the tile, 4 or 2
//
// Blocks pass through LDS twice: as they are stored (buffer_load .. lds, one or two steps ahead, no registers), then
// expanded as above.  Rows of B come straight to registers, half a step (16 rows) at a time and a step ahead,
// and a column group of them is split right before its six instructions.
//
// 128 columns: 8 waves, two per SIMD, with 128 registers of sums.  64 columns: 12 waves with 64 (16 waves, four per
// SIMD, spill; 8 are 3 % slower), and LDS for one step ahead.  Back to back, C handed in, and with fp32 instructions: tiles of 128, 8192 x 8192, 50 % pruned,
// 111 and 133 us, 16384 x 2048, 70 % pruned, 59 and 73; tiles of 64, 4096 x 1024, 70 % pruned, 128 columns, 11.0 and 12.2, 8192 x 8192, 90 % pruned,
// 64 columns, 56 and 68, 8192 x 2048, 50 % pruned, 64 columns, 20 and 23.  At 4096 x 1024 32 steps are three per wave at most.  Up to FEW_STEPS steps the fp32 kernel's
// 16 waves make one each, and stay (4096 x 300: 7.6 and 8.0 us; 8192 x 512: 8.9 both).
//
// What bounds it: on 8192 x 8192 the matrix cores are busy a good third of the time; 11 vector instructions beside each of theirs (192 per 16 rows for B, which
// every panel splits anew, 44 for A) overlap with it only in part, and the power limit holds the clock to 2 GHz.  Splitting B once, in a launch
// of its own, leaves 2.6 vector instructions but moves 6 bytes per value, 19 TB/s through the L2s: 15 % faster, for a workspace that
// spmm_execute does not have.  One wave per SIMD with everything interleaved is slower: a single wave issues an instruction every
// 5 cycles only.  With two, the splitting of the next group placed between the matrix instructions (also over halves and steps)
// takes 4 % fewer cycles and the same time: the clock falls by what the schedule gains.
constexpr int FEW_STEPS = 16;
constexpr int split_waves(int NB) { return NB == 4 ? 8 : 12; }
template <int RUNS, int NB> __global__ __launch_bounds__(64 * split_waves(NB), split_waves(NB) / 4) void spmm_split_tiles_kernel(const tile_args args)
{
    constexpr int W = split_waves(NB), R = 32, NT = NB * R, KO = 64 / R, KS = OPS * KO;
    constexpr int STAGES = NB == 4 ? 2 : 1;            // blocks on their way to a wave
    typedef typename BVec<NB>::type b_t;
    constexpr int AL = (RUNS * 256 * 6 + 1023) / 1024;  // loads of 1 KiB for one
    constexpr int STAGE_WORDS = 256 * AL, SLOT = A_SLOT_WORDS + STAGES * STAGE_WORDS;
    static_assert(W * SLOT >= W / 2 * NB * Tile<R>::GROUPS * 256, "the sums fit");
    __shared__ __attribute__((aligned(16))) float lds[W * SLOT];
    struct loss {  // bit i: the wave lost bits of B's i-th group of columns; has entries in the panel's i-th row
        uint32_t groups, rows, found;  // found: bits lost 1, sums that are not finite 2
    };
    __shared__ loss losses[W];
    __shared__ uint32_t verdicts[W];

    const uint32_t id = place_in_matrix(args.first), nt = id % (uint32_t)args.n_tiles, panel = id / (uint32_t)args.n_tiles;
    if (panel >= (uint32_t)args.n_panels) return;
    const uint32_t n0 = nt * (uint32_t)NT;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    float *slot = lds + wave * SLOT, *stages = slot + A_SLOT_WORDS;
    f32x4 *expanded = reinterpret_cast<f32x4 *>(slot + TILE_PLACE0 / 4) + lane;
    const uint32_t n_steps = (uint32_t)args.n_steps;
    const uint32_t *off_p = args.offsets + (size_t)panel * (n_steps + 1);
    const uint32_t N = (uint32_t)args.N;
    const uint32_t count = n_steps > (uint32_t)wave ? (n_steps - (uint32_t)wave + W - 1) / W : 0u;  // steps of this wave
    const uint32_t most = (n_steps + W - 1) / W;                                                                    // of any

    f32x16 acc[NB], cor[NB];  // sums of h h; of the other products
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = cor[j] = f32x16{};
    uint32_t lost = 0, entries = 0;  // of the lane's columns of B; of its row of A
    auto clear = [&] {
#pragma unroll
        for (int q = 0; q < OPS / 4; ++q) expanded[64 * q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    clear();

    // Runs of 64 steps: lane i holds the bounds of the i-th block of the run.  (Loaded inside of the pipeline
    // they would make every step wait for all loads on their way.)
    uint32_t lo = 0, hi = 0, last = 0;
    uint32_t n_in[STAGES];  // entries of the blocks in the stages
    auto bounds = [&](uint32_t first) {
        last = first + 64u < count ? first + 64u : count;
        const uint32_t s = (uint32_t)wave + W * (first + (uint32_t)lane);
        lo = s < n_steps ? off_p[s] : 0u;
        hi = s < n_steps ? off_p[s + 1] : 0u;
    };
    // The compiler knows of these loads and of those of B and counts its waits by both: every step makes the
    // same number of them, in this order (no load passes the empty asm).
    auto fetch_a = [&](uint32_t i, int st) {  // nothing past the run
        const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)(i & 63u));
        const uint32_t units = i < last ? (uint32_t)__builtin_amdgcn_readlane((int)hi, (int)(i & 63u)) - a : 0u;
        n_in[st] = 8u * units;
        const char *block = reinterpret_cast<const char *>(args.stream) + (size_t)a * 48u;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(block), (short)0, (int)(units * 48u), 0x00020000);
        load_to_lds<AL>(r, stages + st * STAGE_WORDS, lane);
        asm volatile("" ::: "memory");
    };
    // Every entry of the stage to its place in the expanded block, which is all zeros at this point; what lies
    // behind the last one to the dump word.  All reads first: one wait for LDS and not one per run.
    auto scatter = [&](int st) {
        f32x4 v[RUNS];
        u32x2 place[RUNS];
        const uint32_t n = n_in[st];
        const float *stage = stages + st * STAGE_WORDS;
        const char *places = reinterpret_cast<const char *>(stage) + n * 4u;
#pragma unroll
        for (int q = 0; q < RUNS; ++q) {
            v[q] = *reinterpret_cast<const f32x4 *>(stage + 4 * lane + 256 * q);
            place[q] = *reinterpret_cast<const u32x2 *>(places + 8 * lane + 512 * q);
        }
        char *cslot = reinterpret_cast<char *>(slot);
#pragma unroll
        for (int q = 0; q < RUNS; ++q) {
            const bool in = (uint32_t)lane * 4u + 256u * (uint32_t)q < n;
            const u32x2 p = u32x2{in ? place[q][0] : 0u, in ? place[q][1] : 0u};
#pragma unroll
            for (int x = 0; x < 4; ++x) *reinterpret_cast<float *>(cslot + ((p[x / 2] >> (16 * (x % 2))) & 0xFFFFu)) = v[q][x];
        }
        lds_in_order();
    };
    // Rows of B from step s on
    auto b_rsrc = [&](uint32_t s) {
        const uint64_t skip = ((uint64_t)s * KS * N + n0) * 4u;
        const uint64_t left = args.b_bytes > skip ? args.b_bytes - skip : 0u;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(args.B)) + skip, (short)0,
                                                 (int)(left > 0xFFFFFFFCull ? 0xFFFFFFFCu : (uint32_t)left), 0x00020000);
    };
    const uint32_t lane_off = ((uint32_t)(lane / R) * N + (uint32_t)(NB * (lane % R))) * 4u, op_pitch = (uint32_t)KO * N * 4u;
    b_t b[2][8];  // halves of a step
    auto fetch_b = [&](__amdgpu_buffer_rsrc_t r, int half) {  // no rows past the last step
        uint32_t off = lane_off + (uint32_t)(8 * half) * op_pitch;
        asm volatile("" : "+v"(off));  // one address register, not one per row
#pragma unroll
        for (int t = 0; t < 8; ++t, off += op_pitch) b[half][t] = buffer_load<NB>(r, off);
        asm volatile("" ::: "memory");
    };
    auto values_of_a = [&](int half, float (&x)[8]) {
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = expanded[64 * (2 * half + t / 4)][t % 4];
#pragma unroll
        for (int q = 0; q < 2; ++q) expanded[64 * (2 * half + q)] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto multiply_parts = [&](__amdgpu_buffer_rsrc_t next, int half) {
        float x[8];
        values_of_a(half, x);
        parts a = in_parts<false>(x, entries);
        const u32x4 h = __builtin_bit_cast(u32x4, a.h);
        entries |= h[0] | h[1] | h[2] | h[3];
        parts_done(a, entries);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 8; ++t) x[t] = part(b[half][t], j);
            // not before this point: two groups of parts do not fit the registers
            asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]));
            parts p = in_parts<true>(x, lost);
            parts_done(p, lost);
            if (j == NB - 1) fetch_b(next, half);
            cor[j] = Tile<R>::mfma(p.l, a.h, cor[j]);
            cor[j] = Tile<R>::mfma(p.h, a.l, cor[j]);
            cor[j] = Tile<R>::mfma(p.m, a.m, cor[j]);
            cor[j] = Tile<R>::mfma(p.m, a.h, cor[j]);
            cor[j] = Tile<R>::mfma(p.h, a.m, cor[j]);
            acc[j] = Tile<R>::mfma(p.h, a.h, acc[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto multiply_whole = [&](__amdgpu_buffer_rsrc_t next, int half) {
        float x[8];
        values_of_a(half, x);
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[j] = Tile<R>::mfma(part(b[half][t], j), x[t], acc[j]);
        fetch_b(next, half);
    };
    auto all_steps = [&](auto multiply_half) {
        for (uint32_t first = 0; first < count; first = last) {
            bounds(first);
            fetch_a(first, 0);
            if (STAGES == 2) fetch_a(first + 1, 1);
            fetch_b(b_rsrc((uint32_t)wave + W * first), 0);
            fetch_b(b_rsrc((uint32_t)wave + W * first), 1);
            for (uint32_t i = first; i < last; i += STAGES) {
#pragma unroll
                for (int u = 0; u < STAGES; ++u) {
                    if (u == 1 && i + 1 >= last) break;
                    first_if_behind(count - i - (uint32_t)u, most);
                    // the step's block has arrived: younger are the other stage's and 16 loads of B
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((STAGES - 1) * AL + 16) : "memory");
                    scatter(u);
                    fetch_a(i + (uint32_t)(u + STAGES), u);
                    const __amdgpu_buffer_rsrc_t next = b_rsrc((uint32_t)wave + W * (i + (uint32_t)u + 1u));
                    multiply_half(next, 0);
                    multiply_half(next, 1);
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no block on its way to the stages
        }
    };
    all_steps(multiply_parts);

    float not_finite = 0.0f;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        acc[j] += cor[j];
#pragma unroll
        for (int x = 0; x < 16; ++x) not_finite = __builtin_fmaf(acc[j][x], 0.0f, not_finite);
    }
    const uint64_t lossy = __ballot((lost & 0xFFFFu) != 0), filled = __ballot(entries != 0), bad = __ballot(not_finite != 0.0f);
    if (lane == 0) losses[wave] = loss{(uint32_t)(lossy | lossy >> 32), (uint32_t)(filled | filled >> 32), (uint32_t)(lossy != 0) + 2u * (uint32_t)(bad != 0)};
    auto none = [](uint32_t, const f32x4 &) {};
    const int one = lane < W ? lane : 0;
    uint32_t found;
    add_halves<R, NB, W>(acc, lds, wave, lane, [&] { found = losses[one].found; });
    if (__builtin_expect(!__any(found != 0), 1)) {
        store_sum<R, NB, W>(args, lds, panel, n0, wave, lane, none);
        return;
    }
    if (!__any(found > 1)) {
        uint32_t groups = 0, rows = 0;
        for (int w = 0; w < W; ++w) {
            groups |= losses[w].groups;
            rows |= losses[w].rows;
        }
        const float enough = args.largest * (float)args.K * 0x1p-101f;  // (infinite: no sum is)
        const bool row = (rows >> (lane % R) & 1) != 0;
        bool small = false;
        store_sum<R, NB, W>(args, lds, panel, n0, wave, lane, [&](uint32_t n, const f32x4 &sum) {
#pragma unroll
            for (uint32_t x = 0; x < 4; ++x)
                small |= row && (groups >> ((n + x - n0) / NB) & 1) != 0 && n + x < N && !(__builtin_fabsf(sum[(int)x]) > enough);
        });
        const bool any_small = __any(small);
        if (lane == 0) verdicts[wave] = any_small;
        __syncthreads();
        if (!__any(verdicts[one] != 0)) return;
    }
    clear();
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = f32x16{};
    all_steps(multiply_whole);
    add_halves<R, NB, W>(acc, lds, wave, lane, [] {});
    store_sum<R, NB, W>(args, lds, panel, n0, wave, lane, none);
}

template <int RUNS, int NB> hipError_t launch_split(tile_args &a, hipStream_t s)
{
    a.n_tiles = (int32_t)(((int64_t)a.N + 32 * NB - 1) / (32 * NB));
    return launch_places(spmm_split_tiles_kernel<RUNS, NB>, a, 64 * split_waves(NB), s);
}
template <int NB> hipError_t launch_split(tile_args &a, int runs, hipStream_t s)
{
    if (runs == 1) return launch_split<1, NB>(a, s);
    if (runs == 2) return launch_split<2, NB>(a, s);
    if (runs == 3) return launch_split<3, NB>(a, s);
    return launch_split<4, NB>(a, s);
}

// ---------------------------------------------------------------- executor, narrow panels

// v + v turned within every row of 16 lanes (CTRL: a DPP row rotation)
template <int CTRL> __device__ __forceinline__ float add_turned(float v)
{
    return v + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}

// The loads before this point start before the work after it and in this order: the compiler would move
// them to their first use, and count the wait for a block's entries by the wrong loads.
__device__ __forceinline__ void keep_loads_here() { __builtin_amdgcn_sched_barrier(0); }

// One workgroup computes a tile of C: a panel of 8 rows x 4 * NB columns, with v_mfma_f32_4x4x1 (16
// products of 4 rows by 4 columns, one column of A each): 16 columns of A per instruction.  An operand of B
// is then 16 rows x 4 columns of B as they lie in memory, so B needs no LDS, both row groups use it, and
// B of 4 or 8 columns leaves no part of an instruction idle; panels of 8 rows give a matrix of 2048 rows
// 256 workgroups, where panels of 16 leave half the chip without work.
//
// W       waves of the workgroup, cutting K as in the kernel above
// AL      16-byte loads per lane that hold any block of the plan (256 entries each)
// WIDE    64-bit addresses of B, word by word
//
// What bounds it: with four columns the plan's bytes (2048 x 8192, 70 % pruned: 30 MB in 7.1 us, 2.6 us of them
// the launch; chunks 15.8, panels of 16 rows 17.1), with sixteen the vector ALUs, which the matrix
// instructions share (9 to 11 cycles each, measured, of the nominal 8, and 30 to 40 others per step), and the vector L1 (busy
// 57 %): 10.0 us; chunks 21.4, panels of 16 rows 17.2.  Where a block has 256 entries or fewer, writing zeros to its places
// is cheaper than clearing all of it (8192 x 8192, 90 % pruned, 4 columns: 14.7 -> 12.3 us).  Asking for blocks
// two steps ahead, or sixteen waves, changed nothing; panels of 16 rows of this kind gain 15 % at 8192 rows
// with 16 columns and lose as much or more elsewhere.
template <int NB, int W, int AL, bool WIDE, int MINW>
__global__ __launch_bounds__(64 * W, MINW) void spmm_narrow_tiles_kernel(const tile_args args)
{
    typedef typename BVec<NB>::type bvec_t;
    constexpr int R = NARROW_ROWS;
    constexpr int KS = 1024 / R;      // columns of A per step
    constexpr int H = KS / 16;        // operands of B per step
    constexpr int G = R / 4;          // row groups
    constexpr int NT = NB * 4;        // columns of C per tile
    constexpr int SLOT = A_SLOT_WORDS;
    constexpr int T = R * NB;         // sums per lane
    static_assert(R * NT <= SLOT, "a wave's sums fit its slot");
    __shared__ __attribute__((aligned(16))) float lds[W * SLOT];

    const uint32_t id = place_in_matrix(args.first), nt = id % (uint32_t)args.n_tiles, panel = id / (uint32_t)args.n_tiles;
    if (panel >= (uint32_t)args.n_panels) return;
    const uint32_t n0 = nt * (uint32_t)NT;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    float *slot = lds + wave * SLOT;
    char *cslot = reinterpret_cast<char *>(slot);
    f32x4 *expanded = reinterpret_cast<f32x4 *>(slot + TILE_PLACE0 / 4) + lane;
    const uint32_t n_steps = (uint32_t)args.n_steps;
    const uint32_t *off_p = args.offsets + (size_t)panel * (n_steps + 1);
    const uint32_t N = (uint32_t)args.N;
    const uint32_t count = n_steps > (uint32_t)wave ? (n_steps - (uint32_t)wave + W - 1) / W : 0u;  // steps of this wave

    f32x4 acc[G][NB];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int c = 0; c < NB; ++c) acc[g][c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < OPS / 4; ++q) expanded[64 * q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // lane l: columns NB * (l % 4) .. of row l / 4 of the operand
    bvec_t b[H];
    auto fetch_b = [&](uint32_t i, int h) {  // no rows past the last step
        const uint32_t s = (uint32_t)wave + W * i;
        if constexpr (WIDE) {
            const uint64_t row = (uint64_t)s * KS + (uint32_t)(16 * h + lane / 4);
            const float *p = args.B + (row < (uint64_t)args.K ? row : (uint64_t)args.K - 1u) * N;
#pragma unroll
            for (int j = 0; j < NB; ++j) {  // rows and columns outside B repeat its last ones (never used)
                const uint32_t n = n0 + (uint32_t)(NB * (lane % 4) + j);
                b[h][j] = p[n < N ? n : N - 1u];
            }
        } else {
            const uint64_t skip = ((uint64_t)s * KS * N + n0) * 4u;
            const uint64_t left = args.b_bytes > skip ? args.b_bytes - skip : 0u;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(args.B)) + skip, (short)0,
                                                                               (int)(left > 0xFFFFFFFCull ? 0xFFFFFFFCu : (uint32_t)left), 0x00020000);
            b[h] = buffer_load<NB>(r, ((uint32_t)(lane / 4) * N + (uint32_t)(NB * (lane % 4))) * 4u + (uint32_t)h * (64u * N));
        }
    };
    // Runs of 64 steps: lane i holds the bounds of the i-th block of the run.  (With the bounds loaded
    // inside of the pipeline every step would have to wait for all loads on their way, in case this one
    // is among them; for the same reason all steps make the same number of loads, up to 512 entries.)
    uint32_t lo = 0, hi = 0, last = 0, n_next = 0;
    f32x4 va[AL];
    u32x2 vp[AL];
    auto fetch_a = [&](uint32_t i) {
        const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)lo, (int)(i & 63u));
        n_next = i < last ? 8u * ((uint32_t)__builtin_amdgcn_readlane((int)hi, (int)(i & 63u)) - a) : 0u;
        const char *block = reinterpret_cast<const char *>(args.stream) + (size_t)a * 48u;
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(block), (short)0, (int)(n_next * 4u), 0x00020000);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(block) + (size_t)n_next * 4u, (short)0, (int)(n_next * 2u), 0x00020000);
#pragma unroll
        for (int q = 0; q < AL; ++q) {
            if (AL > 2 && q > 0 && n_next <= 256u) break;  // few blocks are as long as the longest where rows are uneven
            va[q] = buffer_load<4>(rv, (uint32_t)lane * 16u + 1024u * (uint32_t)q);
            vp[q] = __builtin_amdgcn_raw_buffer_load_b64(rp, (int)((uint32_t)lane * 8u + 512u * (uint32_t)q), 0, 0);
        }
    };

    for (uint32_t first = 0; first < count; first = last) {
        last = first + 64u < count ? first + 64u : count;
        {
            const uint32_t s = (uint32_t)wave + W * (first + (uint32_t)lane);
            lo = s < n_steps ? off_p[s] : 0u;
            hi = s < n_steps ? off_p[s + 1] : 0u;
        }
        fetch_a(first);
        keep_loads_here();
#pragma unroll
        for (int h = 0; h < H; ++h) fetch_b(first, h);
        keep_loads_here();
        for (uint32_t i = first; i < last; ++i) {
            // ---- the block's entries go to their places in the expanded block, zero otherwise
            const uint32_t n = n_next;
            u32x2 places[AL];
#pragma unroll
            for (int q = 0; q < AL; ++q) places[q] = vp[q];
            auto scatter = [&](auto value) {
#pragma unroll
                for (int q = 0; q < AL; ++q)
                    if (q == 0 || n > 256u * (uint32_t)q)
                        if ((uint32_t)lane * 4u + 256u * (uint32_t)q < n)
#pragma unroll
                            for (int x = 0; x < 4; ++x)
                                *reinterpret_cast<float *>(cslot + ((places[q][x / 2] >> (16 * (x % 2))) & 0xFFFFu)) = value(q, x);
            };
            scatter([&](int q, int x) { return va[q][x]; });
            lds_in_order();
            fetch_a(i + 1);
            keep_loads_here();
            f32x4 a[OPS / 4];
#pragma unroll
            for (int q = 0; q < OPS / 4; ++q) a[q] = expanded[64 * q];
            // ---- zeros again for the next block, at its places where they are few
            if (AL <= 2 || n <= 256u) {
                lds_in_order();
                scatter([](int, int) { return 0.0f; });
            } else {
#pragma unroll
                for (int q = 0; q < OPS / 4; ++q) expanded[64 * q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
#pragma unroll
            for (int h = 0; h < H; ++h) {
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int c = 0; c < NB; ++c)
                        acc[g][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(a[(h * G + g) / 4][(h * G + g) % 4], part(b[h], c), acc[g][c], 0, 0, 0);
                fetch_b(i + 1, h);
            }
        }
    }

    // ---- add the 16 products of an instruction: halves, then quarters of the wave, each keeping half of
    //      the sums, then within rows of 16 lanes
    float v[T];  // row q / NB, columns NB * (lane % 4) + q % NB
#pragma unroll
    for (int q = 0; q < T; ++q) v[q] = acc[q / NB / 4][q % NB][q / NB % 4];
#pragma unroll
    for (int q = 0; q < T / 2; ++q) {
        const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[q]), __float_as_uint(v[q + T / 2]), false, false);
        v[q] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
#pragma unroll
    for (int q = 0; q < T / 4; ++q) {
        const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[q]), __float_as_uint(v[q + T / 4]), false, false);
        v[q] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
    }
#pragma unroll
    for (int q = 0; q < T / 4; ++q) v[q] = add_turned<0x124>(add_turned<0x128>(v[q]));
    if (lane % 16 < 4) {
        const int o = T / 2 * (lane / 32) + T / 4 * (lane / 16 % 2);
#pragma unroll
        for (int q = 0; q < T / 4; ++q) slot[(o + q) / NB * NT + NB * (lane % 4) + (o + q) % NB] = v[q];
    }
    // ---- add the waves' tiles, in order
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < (uint32_t)(R * NT); t += 64 * W) {
        const uint32_t row = panel * (uint32_t)R + t / NT, n = n0 + t % NT;
        float sum = lds[t];
#pragma unroll
        for (int u = 1; u < W; ++u) sum += lds[u * SLOT + t];
        if (row < (uint32_t)args.M && n < N) args.C[(size_t)row * N + n] = sum;
    }
}

template <int NB, int W, int AL, bool WIDE, int MINW> hipError_t launch_narrow(tile_args &a, hipStream_t s)
{
    a.n_tiles = (int32_t)(((int64_t)a.N + NB * 4 - 1) / (NB * 4));
    return launch_places(spmm_narrow_tiles_kernel<NB, W, AL, WIDE, MINW>, a, 64 * W, s);
}
template <int NB, int W> hipError_t launch_narrow(tile_args &a, int loads, hipStream_t s)
{
    if (loads == 1) return launch_narrow<NB, W, 1, false, 4>(a, s);
    if (loads == 2) return launch_narrow<NB, W, 2, false, 4>(a, s);
    return launch_narrow<NB, W, 4, false, NB < 4 ? 4 : 2>(a, s);
}
template <int NB> hipError_t launch_narrow(tile_args &a, int waves, int loads, hipStream_t s)
{
    return waves == 8 ? launch_narrow<NB, 8>(a, loads, s) : launch_narrow<NB, 4>(a, loads, s);
}

// Column groups and waves of a workgroup.  While the workgroups of a narrower tile still all find an idle
// compute unit, that tile; then the tile that takes all columns.  Eight waves share the panel where
// its steps give each of them four or more and the workgroups are too few to keep enough waves on
// the chip otherwise.  (1024 x 4096 with 90 % pruned, 16 columns: 4.8 us with tiles of 8, 5.6 us with tiles of
// 16; 2048 x 8192 with 70 % pruned, 4 columns: 7.1 us with eight waves, 9.5 us with four; 4096 x 1024: 3.8 and 3.6 us.)
int narrow_columns(int64_t panels, int64_t N)
{
    int NB = N <= 16 ? 1 : N <= 32 ? 2 : 4;  // a quarter of a row of B at least: of shorter parts the L1 fetches too much beside them
    while (NB < 4 && NB * 4 < N && panels * ((N + NB * 4 - 1) / (NB * 4)) > 256) NB *= 2;
    return NB;
}
int narrow_waves(int64_t panels, int64_t steps, int64_t N, int NB)
{
    return steps >= 32 && panels * ((N + NB * 4 - 1) / (NB * 4)) < (NB == 1 ? 1024 : 512) ? 8 : 4;
}

// ---------------------------------------------------------------- builder

struct position {
    uint32_t step, op, lane;
};
template <int R> __device__ __forceinline__ position position_of(uint32_t row, uint32_t col)
{
    constexpr uint32_t KO = 64 / R, KS = OPS * KO;
    if constexpr (R == NARROW_ROWS) return position{col / KS, col % KS / 16 * (R / 4) + row % R / 4, col % 16 * 4 + row % 4};
    return position{col / KS, col % KS / KO, row % R + R * (col % KO)};
}

enum { BAD_COLUMN = 1, TWICE = 2 };

// Sizes, as bits, between which a value is the sum of its parts (in_parts): 2^-110, the smallest whose last bit is a bf16, and
// 2^128 - 2^119, which rounds to no bf16.
constexpr uint32_t SMALLEST_IN_PARTS = (127u - 110u) << 23, LARGEST_IN_PARTS = 0x7F7F8000u;

// The order of a block's entries.  A wave writes up to 64 of them to LDS at a time, so entries
// that lie in different banks should follow each other: the places of a block fall into 64 classes of
// 16 (place in words modulo 64), and the block takes the first entry of every class, in class order, then the
// second of every class, and so on.  (In the order of the rows, a dense row's entries met in one bank: 2048 x 8192
// with Zipf rows, 90 % pruned, 4 columns took 12.6 us instead of 6.1.)
struct bank {
    uint32_t of, rank_bit;  // the class; the place's number in it
};
__device__ __forceinline__ bank bank_of(const position &p) { return bank{p.lane % 16 * 4 + p.op % 4, p.lane / 16 * 4 + p.op / 4}; }

constexpr int MASK_WORDS = 32;  // bitmap of a block while the plan is built: 16 bits per class
struct block_order {            // of the entries that are the r-th of their classes:
    uint64_t classes[16];       // the classes
    uint16_t first[16];         // how many entries come before them
};

// Where the j-th entry of a block of n (a multiple of eight) entries is stored: lane l of the wave
// reads entries 4 l .. 4 l + 3 of a run of 256 and writes the first of each lane together, then the second.
__device__ __forceinline__ uint32_t stored_at(uint32_t j, uint32_t n)
{
    const uint32_t run = j / 256u * 256u, lanes = (n - run < 256u ? n - run : 256u) / 4u;
    return run + (j - run) % lanes * 4u + (j - run) / lanes;
}

// One wave per row: sets the entries' bits.
template <int R, typename Col> __global__ __launch_bounds__(256) void mark_kernel(const int32_t *row_ptr, const Col *col_idx, int64_t M, int64_t K, int64_t n_steps,
                                                                    uint32_t *masks, uint32_t *flags)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (row >= M) return;
    uint32_t bad = 0;
    for (int64_t q = row_ptr[row] + (int64_t)(threadIdx.x & 63); q < row_ptr[row + 1]; q += 64) {
        const int32_t c = (int32_t)col_idx[q];
        if (c < 0 || (int64_t)c >= K) {
            bad |= BAD_COLUMN;
            continue;
        }
        const position p = position_of<R>((uint32_t)row, (uint32_t)c);
        const bank k = bank_of(p);
        uint32_t *word = masks + ((size_t)(row / R) * n_steps + p.step) * MASK_WORDS + k.of / 2;
        const uint32_t bit = 1u << (k.of % 2 * 16 + k.rank_bit);
        if (atomicOr(word, bit) & bit) bad |= TWICE;
    }
    if (bad) atomicOr(flags, bad);
}

// One wave per block: its length, to offsets[panel][step] in units of eight entries, and its order.
__global__ __launch_bounds__(256) void measure_kernel(const uint32_t *masks, int64_t n_panels, int64_t n_steps, block_order *order,
                                                      uint32_t *counts, uint32_t *offsets, uint32_t *longest)
{
    const int64_t b = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (b >= n_panels * n_steps) return;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t mine = __builtin_popcount(masks[(size_t)b * MASK_WORDS + lane / 2] >> (lane % 2 * 16) & 0xFFFFu);
    uint32_t n = 0;
    for (uint32_t r = 0; r < 16; ++r) {
        const uint64_t classes = __ballot(mine > r);
        if (lane == r) {
            order[b].classes[r] = classes;
            order[b].first[r] = (uint16_t)n;
        }
        n += (uint32_t)__builtin_popcountll(classes);
    }
    if (lane != 0) return;
    counts[b] = n;
    if (n > *longest) atomicMax(longest, n);
    offsets[b / n_steps * (n_steps + 1) + b % n_steps] = (n + 7) / 8;
}

// Exclusive sums of `n` values of 256 threads' shares; returns the total.
__device__ uint64_t scan_block(uint64_t v, uint64_t &before)
{
    __shared__ uint64_t sums[256];
    sums[threadIdx.x] = v;
    __syncthreads();
    for (uint32_t d = 1; d < 256; d *= 2) {
        const uint64_t x = threadIdx.x >= d ? sums[threadIdx.x - d] : 0;
        __syncthreads();
        sums[threadIdx.x] += x;
        __syncthreads();
    }
    before = sums[threadIdx.x] - v;
    const uint64_t total = sums[255];
    __syncthreads();
    return total;
}

// One workgroup per panel: block lengths -> starts within the panel; the panel's length.
__global__ __launch_bounds__(256) void scan_panel_kernel(int64_t n_steps, uint32_t *offsets, uint64_t *panel_base)
{
    uint32_t *o = offsets + (size_t)blockIdx.x * (n_steps + 1);
    uint64_t done = 0;
    for (int64_t s0 = 0; s0 < n_steps; s0 += 256) {
        const int64_t s = s0 + threadIdx.x;
        const uint64_t v = s < n_steps ? o[s] : 0;
        uint64_t before;
        const uint64_t total = scan_block(v, before);
        if (s < n_steps) o[s] = (uint32_t)(done + before);
        done += total;
    }
    if (threadIdx.x == 0) {
        o[n_steps] = (uint32_t)done;
        panel_base[blockIdx.x] = done;
    }
}

// The three kernels above in one, for panels whose bitmaps fit LDS: a workgroup per panel sets the bits there,
// orders the blocks and adds up their lengths.  (4096 x 4096, 80 % pruned, panels of 16 rows: the bits alone, an atomic
// operation in global memory for every entry, took most of 150 us; the three together now take 22.)
constexpr int64_t MOST_STEPS_IN_LDS = 1024;  // 128 KiB of bitmaps; one step per thread while the lengths are added
template <int R, typename Col> __global__ __launch_bounds__(1024) void panel_kernel(const int32_t *row_ptr, const Col *col_idx, int64_t M, int64_t K, int32_t n_steps,
                                                                      uint32_t *masks, block_order *order, uint32_t *counts, uint32_t *offsets,
                                                                      uint64_t *panel_base, uint32_t *flags, uint32_t *longest)
{
    extern __shared__ uint32_t bits[];
    __shared__ uint32_t units[1024], sums[16];
    constexpr int WAVES = 16, PER_ROW = R < WAVES ? WAVES / R : 1;  // waves per row
    const int64_t panel = blockIdx.x;
    const int wave = (int)(threadIdx.x / 64), lane = (int)(threadIdx.x & 63);
    for (int32_t i = (int32_t)threadIdx.x; i < n_steps * MASK_WORDS; i += 1024) bits[i] = 0;
    __syncthreads();
    uint32_t bad = 0;
    for (int r = wave / PER_ROW; r < R; r += WAVES / PER_ROW) {
        const int64_t row = panel * R + r;
        if (row >= M) break;
        for (int64_t q = row_ptr[row] + (int64_t)(wave % PER_ROW * 64 + lane); q < row_ptr[row + 1]; q += 64 * PER_ROW) {
            const int32_t c = (int32_t)col_idx[q];
            if (c < 0 || (int64_t)c >= K) {
                bad |= BAD_COLUMN;
                continue;
            }
            const position p = position_of<R>((uint32_t)row, (uint32_t)c);
            const bank k = bank_of(p);
            const uint32_t bit = 1u << (k.of % 2 * 16 + k.rank_bit);
            if (atomicOr(&bits[p.step * MASK_WORDS + k.of / 2], bit) & bit) bad |= TWICE;
        }
    }
    if (bad) atomicOr(flags, bad);
    __syncthreads();
    uint32_t most = 0;
    for (int32_t s = wave; s < n_steps; s += WAVES) {
        const int64_t b = panel * n_steps + s;
        const uint32_t mask = bits[s * MASK_WORDS + lane / 2], mine = __builtin_popcount(mask >> (lane % 2 * 16) & 0xFFFFu);
        if (lane % 2 == 0) masks[(size_t)b * MASK_WORDS + lane / 2] = mask;
        uint32_t n = 0;
        uint64_t my_classes = 0;
        uint32_t my_first = 0;
#pragma unroll 4
        for (int r = 0; r < 16; ++r) {
            const uint64_t classes = __ballot(mine > (uint32_t)r);
            if (lane == r) {
                my_classes = classes;
                my_first = n;
            }
            n += (uint32_t)__builtin_popcountll(classes);
        }
        if (lane < 16) {
            order[b].classes[lane] = my_classes;
            order[b].first[lane] = (uint16_t)my_first;
        }
        if (lane == 0) {
            counts[b] = n;
            units[s] = (n + 7) / 8;
        }
        most = n > most ? n : most;
    }
    if (lane == 0 && most > *longest) atomicMax(longest, most);
    __syncthreads();
    // thread s: the length of step s, then the sum up to it
    const uint32_t mine = (int32_t)threadIdx.x < n_steps ? units[threadIdx.x] : 0u;
    uint32_t sum = mine;
    for (int d = 1; d < 64; d *= 2) {
        const uint32_t below = __shfl_up(sum, d);
        if (lane >= d) sum += below;
    }
    if (lane == 63) sums[wave] = sum;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int w = 0; w < WAVES; ++w) {
        before += w < wave ? sums[w] : 0u;
        total += sums[w];
    }
    uint32_t *o = offsets + (size_t)panel * ((size_t)n_steps + 1);
    if ((int32_t)threadIdx.x < n_steps) o[threadIdx.x] = before + sum - mine;
    if (threadIdx.x == 0) {
        o[n_steps] = total;
        panel_base[panel] = total;
    }
}

// The sizes of the values: range[0] = the largest, as bits; range[1] = 2^32 less the smallest that is not zero
// (maxima on cleared memory).  Sizes order as their bits do, infinite and NaN ones last.  Few workgroups and one pair of atomics
// from each: two thousand pairs on one address held up a creation of 0.76 ms by 0.06.
__global__ __launch_bounds__(1024) void range_kernel(const float *vals, int64_t nnz, uint32_t *range)
{
    __shared__ uint32_t of_wave[2][16];
    uint32_t largest = 0, smallest = 0;
    auto take = [&](float v) {
        const uint32_t size = __float_as_uint(v) & 0x7FFFFFFFu;
        largest = size > largest ? size : largest;
        smallest = 0u - size > smallest ? 0u - size : smallest;
    };
    const int64_t quads = nnz / 4, first = (int64_t)blockIdx.x * 1024 + threadIdx.x, all = (int64_t)gridDim.x * 1024;
    for (int64_t i = first; i < quads; i += all) {
        const f32x4 v = reinterpret_cast<const f32x4 *>(vals)[i];
        for (int x = 0; x < 4; ++x) take(v[x]);
    }
    for (int64_t i = 4 * quads + first; i < nnz; i += all) take(vals[i]);
    auto over_lanes = [&](int lanes) {
        for (int d = lanes / 2; d > 0; d /= 2) {
            const uint32_t l = __shfl_xor(largest, d), s = __shfl_xor(smallest, d);
            largest = l > largest ? l : largest;
            smallest = s > smallest ? s : smallest;
        }
    };
    over_lanes(64);
    if (threadIdx.x % 64 == 0) {
        of_wave[0][threadIdx.x / 64] = largest;
        of_wave[1][threadIdx.x / 64] = smallest;
    }
    __syncthreads();
    largest = of_wave[0][threadIdx.x % 16];
    smallest = of_wave[1][threadIdx.x % 16];
    over_lanes(16);
    if (threadIdx.x == 0) {
        atomicMax(&range[0], largest);
        atomicMax(&range[1], smallest);
    }
}

// One workgroup: panel lengths -> panel starts; panel_base[n_panels] = length of everything.
__global__ __launch_bounds__(256) void scan_all_kernel(int64_t n_panels, uint64_t *panel_base)
{
    uint64_t done = 0;
    for (int64_t p0 = 0; p0 < n_panels; p0 += 256) {
        const int64_t p = p0 + threadIdx.x;
        const uint64_t v = p < n_panels ? panel_base[p] : 0;
        uint64_t before;
        const uint64_t total = scan_block(v, before);
        if (p < n_panels) panel_base[p] = done + before;
        done += total;
    }
    if (threadIdx.x == 0) panel_base[n_panels] = done;
}

// One thread per block: its final start; the entries that fill up its last group of eight
// (value 0 to the dump place).
__global__ __launch_bounds__(256) void place_kernel(int64_t n_panels, int64_t n_steps, const uint64_t *panel_base, const uint32_t *counts,
                                                    uint32_t *offsets, char *stream)
{
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= n_panels * n_steps) return;
    const int64_t p = b / n_steps, s = b % n_steps;
    uint32_t *o = offsets + p * (n_steps + 1) + s;
    const uint32_t base = (uint32_t)panel_base[p], start = *o + base, n = counts[b], padded = (n + 7) / 8 * 8;
    *o = start;
    if (s + 1 == n_steps) o[1] += base;
    char *block = stream + (size_t)start * 48;
    for (uint32_t i = n; i < padded; ++i) {
        const uint32_t at = stored_at(i, padded);
        reinterpret_cast<float *>(block)[at] = 0.0f;
        reinterpret_cast<uint16_t *>(block + (size_t)padded * 4)[at] = 0;
    }
}

// One wave per row: the entries to their blocks.
template <int R, typename Col> __global__ __launch_bounds__(256) void fill_kernel(const int32_t *row_ptr, const Col *col_idx, const float *vals, int64_t M,
                                                                    int64_t n_steps, const uint32_t *offsets, const uint32_t *masks,
                                                                    const block_order *order, char *stream)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    if (row >= M) return;
    for (int64_t q = row_ptr[row] + (int64_t)(threadIdx.x & 63); q < row_ptr[row + 1]; q += 64) {
        const position p = position_of<R>((uint32_t)row, (uint32_t)col_idx[q]);
        const uint32_t *o = offsets + row / R * (n_steps + 1) + p.step;
        char *block = stream + (size_t)o[0] * 48;
        const uint32_t n = (o[1] - o[0]) * 8;
        const size_t b = (size_t)(row / R * n_steps + p.step);
        const bank k = bank_of(p);
        const uint32_t in_class = masks[b * MASK_WORDS + k.of / 2] >> (k.of % 2 * 16) & 0xFFFFu;
        const uint32_t r = (uint32_t)__builtin_popcount(in_class & ((1u << k.rank_bit) - 1u));
        const uint32_t i = stored_at(order[b].first[r] + (uint32_t)__builtin_popcountll(order[b].classes[r] & ((1ull << k.of) - 1ull)), n);
        reinterpret_cast<float *>(block)[i] = vals[q];
        reinterpret_cast<uint16_t *>(block + (size_t)n * 4)[i] = (uint16_t)(TILE_PLACE0 + (p.op / 4 * 64 + p.lane) * 16 + p.op % 4 * 4);
    }
}

__global__ __launch_bounds__(256) void clear_kernel(u32x4 *p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = u32x4{0, 0, 0, 0};
}

template <int R> hipError_t build(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, TilePlan &out, int &status)
{
    const int64_t nnz = row_ptr[M], P = out.n_panels, S = out.n_steps;
    const size_t mask_bytes = (size_t)(P * S) * MASK_WORDS * 4;
    hipError_t e;
#define TRY(x) do { e = (x); if (e != hipSuccess) return e; } while (0)
    builder::workshop memory;
    builder::uploader upload;  // (released before the memory)
    const bool staged = upload.begin(K, col_idx, vals, nnz, memory.stream), narrow = staged && upload.narrow_columns();
    const size_t at_ptr = memory.reserve((size_t)(M + 1) * 4), at_col = memory.reserve((size_t)nnz * 4), at_val = memory.reserve((size_t)nnz * 4),
                 at_base = memory.reserve((size_t)(P + 3) * 8), at_masks = memory.reserve(mask_bytes),
                 at_order = memory.reserve((size_t)(P * S) * sizeof(block_order)), at_counts = memory.reserve((size_t)(P * S) * 4);
    // the panels' lengths, the flags and the values' sizes behind them, the masks (which panel_kernel writes whole)
    const size_t zeros = (S <= MOST_STEPS_IN_LDS ? at_masks : at_masks + mask_bytes) - at_base;
    TRY(memory.take());
    int32_t *d_ptr = memory.at<int32_t>(at_ptr), *d_col = memory.at<int32_t>(at_col);
    float *d_val = memory.at<float>(at_val);
    uint32_t *d_masks = memory.at<uint32_t>(at_masks), *d_counts = memory.at<uint32_t>(at_counts);
    block_order *d_order = memory.at<block_order>(at_order);
    TRY(hipMalloc(reinterpret_cast<void **>(&out.d_offsets), (size_t)P * (size_t)(S + 1) * 4));
    uint64_t *base = memory.at<uint64_t>(at_base);
    uint32_t *flags = reinterpret_cast<uint32_t *>(base + P + 1);
    const hipStream_t s = memory.stream;
    const unsigned row_blocks = (unsigned)((M + 3) / 4), block_blocks = (unsigned)((P * S + 3) / 4);
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)std::min<size_t>(4096, zeros / 4096 + 1)), dim3(256), 0, s, memory.at<u32x4>(at_base), (int64_t)(zeros / 16));
    TRY(hipMemcpyWithStream(d_ptr, row_ptr, (size_t)(M + 1) * 4, hipMemcpyHostToDevice, s));
    if (staged) {
        TRY(upload.copy(0, reinterpret_cast<char *>(d_col)));
        if (upload.column_outside()) { status = 2; return hipSuccess; }
    } else {
        TRY(hipMemcpyWithStream(d_col, col_idx, (size_t)nnz * 4, hipMemcpyHostToDevice, s));
    }
    auto with_columns = [&](auto *columns) {
        typedef std::remove_reference_t<decltype(*columns)> Col;
        if (S <= MOST_STEPS_IN_LDS) {
            hipLaunchKernelGGL((panel_kernel<R, Col>), dim3((unsigned)P), dim3(1024), (unsigned)(S * MASK_WORDS * 4), s, d_ptr, columns, M, K, (int32_t)S,
                               d_masks, d_order, d_counts, out.d_offsets, base, flags, flags + 1);
        } else {
            hipLaunchKernelGGL((mark_kernel<R, Col>), dim3(row_blocks), dim3(256), 0, s, d_ptr, columns, M, K, S, d_masks, flags);
            hipLaunchKernelGGL(measure_kernel, dim3(block_blocks), dim3(256), 0, s, d_masks, P, S, d_order, d_counts, out.d_offsets, flags + 1);
            hipLaunchKernelGGL(scan_panel_kernel, dim3((unsigned)P), dim3(256), 0, s, S, out.d_offsets, base);
        }
    };
    if (narrow) with_columns(reinterpret_cast<uint16_t *>(d_col));
    else with_columns(d_col);
    hipLaunchKernelGGL(scan_all_kernel, dim3(1), dim3(256), 0, s, P, base);
    TRY(hipGetLastError());
    if (staged) {
        TRY(upload.copy(1, reinterpret_cast<char *>(d_val)));
    } else {
        TRY(hipMemcpyWithStream(d_val, vals, (size_t)nnz * 4, hipMemcpyHostToDevice, s));  // the kernels run meanwhile
    }
    if (R == 32) {
        hipLaunchKernelGGL(range_kernel, dim3((unsigned)std::min<int64_t>(128, nnz / 4096 + 1)), dim3(1024), 0, s, d_val, nnz, flags + 2);
        TRY(hipGetLastError());
    }
    uint64_t answer[3];
    TRY(hipMemcpyWithStream(answer, base + P, 24, hipMemcpyDeviceToHost, s));
    const uint32_t largest = (uint32_t)answer[2], smallest = 0u - (uint32_t)(answer[2] >> 32);
    std::memcpy(&out.largest, &largest, 4);
    out.exact_parts = largest < LARGEST_IN_PARTS && (smallest == 0 || smallest >= SMALLEST_IN_PARTS);
    const uint32_t bad = (uint32_t)answer[1];
    out.loads = std::max(1, (int32_t)(((uint32_t)(answer[1] >> 32) + 255u) / 256u));
    if (bad & BAD_COLUMN) { status = 2; return hipSuccess; }
    if ((bad & TWICE) || answer[0] >= (1ull << 32)) { status = TILES_NOT_POSSIBLE; return hipSuccess; }
    out.stream_words = (int64_t)answer[0] * 12;
    TRY(hipMalloc(reinterpret_cast<void **>(&out.d_stream), (size_t)std::max<int64_t>(out.stream_words, 4) * 4));
    char *stream = reinterpret_cast<char *>(out.d_stream);
    hipLaunchKernelGGL(place_kernel, dim3((unsigned)((P * S + 255) / 256)), dim3(256), 0, s, P, S, base, d_counts, out.d_offsets, stream);
    if (narrow)
        hipLaunchKernelGGL((fill_kernel<R, uint16_t>), dim3(row_blocks), dim3(256), 0, s, d_ptr, reinterpret_cast<uint16_t *>(d_col), d_val, M, S,
                           out.d_offsets, d_masks, d_order, stream);
    else
        hipLaunchKernelGGL((fill_kernel<R, int32_t>), dim3(row_blocks), dim3(256), 0, s, d_ptr, d_col, d_val, M, S, out.d_offsets, d_masks, d_order, stream);
    TRY(hipGetLastError());
    TRY(memory.give_back());
    TRY(hipStreamSynchronize(s));
    upload.arrived();
#undef TRY
    out.device_bytes = out.stream_words * 4 + P * (S + 1) * 4;
    out.built = true;
    builder::staging.count_plan(1);
    status = 0;
    return hipSuccess;
}

}  // namespace

int spmm_tiles_build(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, int32_t rows, TilePlan &out)
{
    out = TilePlan();
    out.rows = rows;
    const int64_t step = TILE_OPERANDS * 64 / rows;
    out.n_panels = (M + rows - 1) / rows;
    out.n_steps = (K + step - 1) / step;
    // The builder runs a wave per row and per block and a workgroup per panel, 256 threads each; HIP takes
    // fewer than 2^32 threads per launch.
    constexpr int64_t MOST = ((int64_t)1 << 24) - 1;
    if ((M + 3) / 4 > MOST || out.n_panels > MOST || (out.n_panels * out.n_steps + 3) / 4 > MOST) {
        out = TilePlan();
        return TILES_NOT_POSSIBLE;
    }
    int status = 0;
    const hipError_t e = rows == NARROW_ROWS ? build<NARROW_ROWS>(M, K, row_ptr, col_idx, vals, out, status) : rows == 32 ? build<32>(M, K, row_ptr, col_idx, vals, out, status) : build<16>(M, K, row_ptr, col_idx, vals, out, status);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        status = e == hipErrorOutOfMemory ? 3 : 4;
    }
    if (status != 0) spmm_tiles_release(out);
    return status;
}

void spmm_tiles_release(TilePlan &p)
{
    if (p.d_stream) (void)hipFree(p.d_stream);
    if (p.d_offsets) (void)hipFree(p.d_offsets);
    if (p.built) builder::staging.count_plan(-1);
    p = TilePlan();
}

// Fitted; against 600 other products (bench.py --workload paths: 4 to 45 % of the entries kept, 4 to 256 columns)
// the rms error is 4 % for panels of 16 and 32 rows and 11 % for 8.
double spmm_tiles_time(int rows, int64_t M, int64_t K, int64_t N, double density, double peak, int *NB_out)
{
    const int64_t panels = (M + rows - 1) / rows, steps = (K * rows + 1023) / 1024;
    if (rows == NARROW_ROWS) {
        static const double ns_per_step[3] = {30, 61, 85}, ns_density[3] = {120, 114, 145}, us_per_round[3] = {0.02, 0.2, 0.3};
        const int NB = narrow_columns(panels, N), i = NB == 1 ? 0 : NB == 2 ? 1 : 2;
        if (NB_out) *NB_out = NB;
        // Several workgroups share a compute unit: a unit with one more than the others takes
        // about half as much longer.
        const double share = std::max(1.0, (double)(panels * ((N + NB * 4 - 1) / (NB * 4))) / 256.0), rounds = 0.5 * (share + std::ceil(share));
        return 2.6 + rounds * (1e-3 * (double)steps * (ns_per_step[i] + ns_density[i] * density) + us_per_round[i]) +
               1e-3 * (double)steps * ns_density[i] * (peak - density);
    }
    // A compute unit holds one workgroup at a time.
    // R = 16, 32; NB = 1, 2, 4.  (R = 32 with NB = 2 and 4 on bf16 instructions: 8 and 16 % less per step than on fp32 ones.  With
    // few steps NB = 2 runs on fp32 ones: 3 % more than estimated.)
    static const double ns_per_step[2][3] = {{99, 169, 275}, {146, 190, 345}}, us_per_round[2][3] = {{1.36, 1.61, 1.75}, {2.1, 3.6, 4.5}},
                        ns_density[2][3] = {{60, 60, 60}, {60, 100, 130}};
    double best = 0.0;
    for (int i = 0, NB = 1; i < 3; ++i, NB *= 2) {
        if (NB > 1 && rows * NB >= 2 * N) break;  // more than half of the tile idle
        const int64_t blocks = panels * ((N + rows * NB - 1) / (rows * NB));
        const double more = ns_density[rows == 32][i], ns = ns_per_step[rows == 32][i] + more * std::max(0.0, density - 0.1);
        const double t = 1.1 + (double)((blocks + 255) / 256) * (1e-3 * (double)steps * ns + us_per_round[rows == 32][i]) +
                         1e-3 * (double)steps * more * (peak - density);
        if (i == 0 || t < best) {
            best = t;
            if (NB_out) *NB_out = NB;
        }
    }
    return best;
}

uint32_t spmm_tiles_of_set(int rows, int64_t M, int64_t K, int32_t N, int64_t stream_words)
{
    int NB = 1;
    spmm_tiles_time(rows, M, K, N, 0.0, 0.0, &NB);
    const uint32_t tiles = (uint32_t)(((int64_t)N + NB * rows - 1) / (NB * rows));
    const bool wide = (int64_t)TILE_OPERANDS * 64 / rows * 4 * N >= ((int64_t)1 << 32);
    return rows == 16 && !wide ? tiles_of_set(NB * rows, tiles, K, N, stream_words) : tiles;
}

int spmm_tiles_execute(const TilePlan &p, int64_t M, int64_t K, const float *B, int32_t N, float *C, void *stream)
{
    tile_args a{p.d_stream, p.d_offsets, B, C, (uint64_t)K * (uint64_t)N * 4u, (int32_t)p.n_panels, (int32_t)p.n_steps, 1,
                (int32_t)M, (int32_t)K, N, 0, p.largest, 0};
    hipStream_t s = (hipStream_t)stream;
    const int64_t step_bytes = (int64_t)TILE_OPERANDS * 64 / p.rows * 4 * N;  // rows of B a step touches
    if (step_bytes >= ((int64_t)1 << 32))
        return (int)(p.rows == NARROW_ROWS ? launch_narrow<4, 8, 4, true, 2>(a, s)
                     : p.rows == 32        ? launch<32, 4, 8, false, 2, true>(a, s)
                                           : launch<16, 4, 8, false, 2, true>(a, s));
    if (p.rows == NARROW_ROWS) {
        const int NB = narrow_columns(p.n_panels, N), W = narrow_waves(p.n_panels, p.n_steps, N, NB);
        return (int)(NB == 1 ? launch_narrow<1>(a, W, p.loads, s) : NB == 2 ? launch_narrow<2>(a, W, p.loads, s) : launch_narrow<4>(a, W, p.loads, s));
    }
    int NB = 1;
    spmm_tiles_time(p.rows, M, K, N, 0.0, 0.0, &NB);
    switch (p.rows * 8 + NB) {
    case 32 * 8 + 4: return (int)(p.exact_parts ? launch_split<4>(a, p.loads, s) : launch<32, 4, 8, false, 2>(a, s));
    case 32 * 8 + 2: return (int)(p.n_steps <= FEW_STEPS || !p.exact_parts ? launch<32, 2, 16, false, 4>(a, s) : launch_split<2>(a, p.loads, s));
    case 32 * 8 + 1: return (int)launch<32, 1, 16, true, 4>(a, s);
    case 16 * 8 + 4: return (int)launch<16, 4, 8, false, 2>(a, s, p.stream_words);
    case 16 * 8 + 2: return (int)launch<16, 2, 8, true, 2>(a, s, p.stream_words);
    default: return (int)launch<16, 1, 16, true, 4>(a, s, p.stream_words);
    }
}
