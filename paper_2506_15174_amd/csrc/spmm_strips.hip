// gfx950 executor of the strips path: C <- A x B with eight columns of B in LDS at a time (format: spmm_strips.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "spmm_launch.h"
#include "spmm_places.h"
#include "spmm_strips_build.h"
#include "spmm_upload.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef float f32x4_unaligned __attribute__((ext_vector_type(4), aligned(4)));
typedef const uint64_t __attribute__((address_space(4))) scalar_words;  // read through the scalar cache where the address is uniform

struct strip_args {
    const char *stream;
    const u32x2 *units;
    const uint32_t *rows;
    const float *B;
    float *C;
    uint64_t b_bytes;   // bytes of B
    // Strips of all groups (of which a C that fits the device's memory has fewer than 2^30: a place holds 512 bytes of it in
    // bands, and there are 2048 or one per strip without); the launch's first.
    uint32_t n_places, first;
    int32_t K, N, bands, band_rows;
    uint32_t n_units, n_groups, n_strips, set;  // set: strips that come first, of all groups (spmm_strips_of_set)
    uint32_t share;                             // places of an XCD in this launch
};

// v of lane l ^ 1, l ^ 2, l ^ 4 or l ^ 8
template <int CTRL> __device__ __forceinline__ float moved(float v)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
template <int BIT> __device__ __forceinline__ float other(float v)
{
    if constexpr (BIT == 1) return moved<0xB1>(v);              // 1 0 3 2 of four lanes
    if constexpr (BIT == 2) return moved<0x4E>(v);              // 2 3 0 1
    if constexpr (BIT == 4) return moved<0x141>(moved<0x1B>(v));  // eight lanes mirrored, after four lanes mirrored
    if constexpr (BIT == 8) return moved<0x128>(v);             // 16 lanes turned by eight
}
// v + v of lane l ^ 16 or l ^ 32
__device__ __forceinline__ float add_row(float v)
{
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
__device__ __forceinline__ float add_half(float v)
{
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

// One workgroup computes eight columns of C for the rows of one group of units (units g, g + n_groups, ...; unit after
// unit a wave): it copies its strip of B to LDS, and every lane gathers the rows of the strip that its entries name.
//
// BANDS  the strip does not fit LDS: it comes in bands of columns of A, one after the other, and a wave has one unit at most
// WIDE   64-bit addresses of B, word by word: for the few N whose 32 rows span 4 GiB
//
// Why: a gather of rows of B from the vector L1 moves 64 bytes per cycle and compute unit at most (16 cycles per wave load),
// reads of LDS 256 where the lanes' banks differ; and a lane that owns a part of a row adds up by itself, without a
// cross-lane step per entry.  A lane holds four sums per column, for the four steps of a group: chains of a quarter of its
// entries.
//
// Every 12 groups, of whatever bands, they go to a total.  Error against 64 bits and time with and without that, 128 columns:
//   8192 x 8192, 50 % kept                    1.48e-7, 218 us;   4.08e-7, 211 us
//   4096 x 16384, 5 % kept, in four bands     0.94e-7, 47.5 us;  1.40e-7, 47.5 us
//
// What bounds it: LDS (two reads of 4.3 cycles per step and wave, 1.15 times that with the collisions that the builder's order
// leaves), the vector ALUs (8 multiply-adds and 2 others per step) and the fetch of the entries (384 bytes per step) take
// about ten cycles each of the 15 that a step and wave takes of a compute unit; and before them the copy of the strip: the
// vector L1 fetches a line of 128 bytes for 32, 2 cycles, so 4096 rows take 3.6 us.
//
// Three plans in turn (and one back to back), on chunks and on strips:
//   4096 x 4096, 95 % pruned, 128 columns                     17.6 (16.1) -> 12.4 us (11.1)
//   3001 x 2511, 85 % in lognormal rows, 200 columns          37.4 (35.3) -> 17.8 (17.0)
//   8968 x 2473, 92 %, 96 columns                             41.3 (39.2) -> 14.0 (13.2)
//
// One back to back, with the entries' addresses read only when a unit or band begins, waits for all fetches once a round and the
// waves in the order of their age, and as it is now: the second 18.5 -> 17.5 us, the third 14.5 -> 14.2, 8192 x 8192, 95 % in lognormal rows, 64
// columns, in two bands 24.5 -> 23.6, 5376 x 14464, 89 %, 40 columns, in three 39.0 -> 37.2; 28 products 2 % on average, two of them 2 % slower.
// Four or six groups in registers are slower by 1 and 5 %, a third half of a group read ahead from LDS by 1 %.
//
// An accumulator's registers hold columns 1 0 3 2 of its four: a v_fmac of three registers that are all even or all odd takes 4.9
// cycles, else 2.8, and those of LDS hold them in order (1 to 3 % of the product).
template <bool BANDS, bool WIDE> __global__ __launch_bounds__(64 * STRIP_WAVES, STRIP_WAVES / 4) void spmm_strips_kernel(const strip_args args)
{
    extern __shared__ __attribute__((aligned(32))) char lds[];  // (whole rows: the halves of one differ in a bit of the address)
    // Workgroups are dealt to the eight XCDs in turn: each takes an eighth of the places, next to each other, so that the strips of
    // a group, which read the same entries, share an L2, and in two sets (spmm_strips_of_set) half of the XCDs fetch half of B.
    // (The arguments all at once: in rounds, each where it is needed, the last one's wait would come behind the unit's place.)
    asm volatile("" ::"s"(args.units), "s"(args.B), "s"(args.b_bytes), "s"(args.n_places), "s"(args.first), "s"(args.K), "s"(args.N), "s"(args.bands), "s"(args.band_rows),
                 "s"(args.n_units), "s"(args.n_groups), "s"(args.n_strips), "s"(args.set), "s"(args.share));
    const uint32_t place = args.first + blockIdx.x % 8u * args.share + blockIdx.x / 8u;
    if (place >= args.n_places) return;
    const set_place at = place_in_sets(place, args.n_groups, args.n_strips, args.set);
    const uint32_t group = at.row, strip = at.column;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    constexpr int AHEAD = 3;  // groups of a unit in registers: the one at work and the next two
    constexpr int Q = 2;  // fours of columns; the lane reads four i ^ turn of its rows as the i-th
    static_assert(Q * 4 == STRIP_COLS, "the fours of a row change places with one bit");
    const uint32_t turn = (uint32_t)lane % Q, N = (uint32_t)args.N, col0 = strip * STRIP_COLS, band_rows = (uint32_t)args.band_rows;
    const int bands = BANDS ? args.bands : 1;
    const uint32_t own = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)lds + turn * 16u;  // what the lane reads first of row 0

    if (threadIdx.x < Q) *reinterpret_cast<f32x4 *>(lds + band_rows * STRIP_ROW_BYTES + threadIdx.x * 16) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto copy_band = [&](uint32_t band) {
        const uint32_t row0 = band * band_rows, rows = min(band_rows, (uint32_t)args.K - row0);
        if constexpr (WIDE) {
            for (uint32_t t = threadIdx.x; t < rows * Q; t += 64 * STRIP_WAVES) {
                const float *p = args.B + (uint64_t)(row0 + t / Q) * N;
                const uint32_t n = col0 + t % Q * 4;
                f32x4 x;
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) x[c] = n + c < N ? p[n + c] : 0.0f;
                *reinterpret_cast<f32x4 *>(lds + t * 16) = x;
            }
        } else {
            // 1024 bytes at a time, Q lanes a row.  (Past the end of B zeros, past the end of a row what follows: columns that C
            // does not have.)
            const uint32_t off = (uint32_t)(lane / Q) * N * 4u + (uint32_t)(lane % Q) * 16u;
            constexpr uint32_t OP_ROWS = 64 / Q;
            for (uint32_t op = (uint32_t)wave; op * OP_ROWS < rows; op += STRIP_WAVES) {
                const uint64_t skip = ((uint64_t)(row0 + op * OP_ROWS) * N + col0) * 4u, left = args.b_bytes - skip;
                const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(args.B)) + skip, (short)0,
                                                                                   (int)(left > 0xFFFFFFFCull ? 0xFFFFFFFCu : (uint32_t)left), 0x00020000);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(lds + op * 1024), 16, (int)off, 0, 0, 0);
            }
        }
    };
    // A unit's groups in a band (none where there is no unit), asked for when those before them are still to be multiplied.
    struct run {
        uint32_t first, groups;
    };
    auto groups_of = [&](uint32_t unit, uint32_t band) {
        const bool is = unit < args.n_units;
        const uint64_t d = ((scalar_words *)args.units)[(size_t)(is ? unit : 0u) * (uint32_t)bands + band];
        return run{(uint32_t)d, is ? (uint32_t)(d >> 32) : 0u};
    };
    const uint32_t pitch = STRIP_WAVES * args.n_groups;
    uint32_t unit = group + (uint32_t)wave * args.n_groups;
    run next = groups_of(unit, 0);
    copy_band(0);
    bool copied = false;  // the first band, and waited for

    for (;; unit += pitch) {
        const bool any = unit < args.n_units;
        if (!any && copied) break;
        uint32_t word = STRIP_NO_ROW;
        f32x4 acc[STRIP_STEPS][Q], total[Q] = {};  // of the last groups; of all before them
        int rounds = 0;                             // of up to three groups that are in acc, of all bands
        auto collect = [&] {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                total[q] += (acc[0][q] + acc[1][q]) + (acc[2][q] + acc[3][q]);
#pragma unroll
                for (int e = 0; e < STRIP_STEPS; ++e) acc[e][q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            }
        };
#pragma unroll
        for (int e = 0; e < STRIP_STEPS; ++e)
#pragma unroll
            for (int q = 0; q < Q; ++q) acc[e][q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        for (int band = 0; band < bands; ++band) {
            const uint32_t first = next.first, groups = next.groups;
            const char *stream = args.stream + (size_t)first * STRIP_GROUP_BYTES;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(stream), (short)0, (int)(groups * STRIP_GROUP_BYTES), 0x00020000);
            f32x4 values[AHEAD];
            u32x2 places[AHEAD];
            constexpr int LOADS = 2;               // of a fetch
            auto fetch = [&](int k, uint32_t g) {  // nothing past the unit
                values[k] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, (int)(g * STRIP_GROUP_BYTES), 0));
                places[k] = __builtin_amdgcn_raw_buffer_load_b64(r, 1024 + lane * 8, (int)(g * STRIP_GROUP_BYTES), 0);
            };
            // The compiler would move the loads to their first use.
            auto keep_order = [] { __builtin_amdgcn_sched_barrier(0); };
            keep_order();
            fetch(0, 0);
            keep_order();
            fetch(1, 1);
            keep_order();
            next = band + 1 < bands ? groups_of(unit, (uint32_t)band + 1u) : groups_of(unit + pitch, 0u);
            if (BANDS && band > 0) {
                __syncthreads();
                copy_band((uint32_t)band);
                __syncthreads();
            } else if (!copied) {
                // All loads but those of the two fetches, which a barrier of the compiler's would wait for too: the copy's are older than
                // theirs, and none is younger (the build looks whether the compiler kept it so: check_waits_at_barriers).
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * LOADS) : "memory");
            }
            copied = true;
            if (!BANDS || band + 1 == bands) word = args.rows[(size_t)(any ? unit : 0u) * 64u + (uint32_t)lane];
            // (waited for here: in the loop below its wait would be one for all reads of LDS)
            asm volatile("" ::"s"(next.first), "s"(next.groups));
            f32x4 x[2][2][Q];  // rows of the strip: two steps each, read while the other two are multiplied
            auto read = [&](int k, int h) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    // (as an integer, with the strip's address in LDS in what is added anyway: to a pointer the compiler would add
                    // it once more)
                    uint32_t at;
                    if (e == 0) asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(places[k][h]), "n"(STRIP_ROW_BYTES), "v"(own));
                    else asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(at) : "v"(places[k][h]), "n"(STRIP_ROW_BYTES), "v"(own));
#pragma unroll
                    for (int q = 0; q < Q; ++q) x[h][e][q] = *(const lds_f32x4 *)(size_t)(at ^ (uint32_t)q * 16u);
                }
            };
            auto multiply = [&](int k, int h) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int q = 0; q < Q; ++q)
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            f32x4 &to = acc[2 * h + e][q];
                            to[c ^ 1] = __builtin_fmaf(values[k][2 * h + e], x[h][e][q][c], to[c ^ 1]);
                        }
            };
            auto work = [&](int k, bool more) {
                read(k, 1);
                keep_order();
                multiply(k, 0);
                keep_order();
                if (more) read((k + 1) % AHEAD, 0);
                keep_order();
                multiply(k, 1);
                keep_order();
            };
            auto round_ends = [&] {
                // (four registers in a row, not any four)
#pragma unroll
                for (int e = 0; e < STRIP_STEPS; ++e)
#pragma unroll
                    for (int q = 0; q < Q; ++q) asm volatile("" : "+v"(acc[e][q]));
                if (++rounds == 12 / AHEAD) {
                    collect();
                    rounds = 0;
                }
            };
            // Whole rounds first, then what is left of one: a loop that may be left inside of a round makes the compiler wait, at its
            // top, for every fetch but the last.
            __builtin_amdgcn_s_waitcnt(0x0F72);  // all but two loads (of which it would wait for the last in the loop)
            read(0, 0);
            // Of the four waves of a SIMD the one that started first would go first: 9.7, 10.1, 10.8 and 11.5 us at the end of equal units.
            // Of those at their last unit the one that has least of it behind it does, before them those that have another.
            const uint32_t last = unit + pitch >= args.n_units ? groups : ~0u / 4u;
            uint32_t g = 0;
            for (; g + AHEAD <= groups; g += AHEAD) {
                if (g * 4u < last) __builtin_amdgcn_s_setprio(3);
                else if (g * 2u < last) __builtin_amdgcn_s_setprio(2);
                else if (g * 4u < last * 3u) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
#pragma unroll
                for (int k = 0; k < AHEAD; ++k) {
                    fetch((k + 2) % AHEAD, g + (uint32_t)k + 2u);
                    keep_order();
                    work(k, true);
                }
                round_ends();
            }
            if (g < groups) {
                work(0, true);
                if (g + 1 < groups) work(1, false);
                round_ends();
            }
        }
        if (!any) break;
        collect();
        // ---- the sums of the parts of a row: lanes l and l ^ 1 each keep the four that they read first (the other
        // one has it as its second); from then on a lane has one four
#pragma unroll
        for (int q = 0; q < Q; ++q) total[q] = __builtin_shufflevector(total[q], total[q], 1, 0, 3, 2);
        const uint32_t row = word & ((1u << STRIP_PARTS_SHIFT) - 1u);
        const uint32_t parts_log2 = __builtin_amdgcn_readfirstlane(word >> STRIP_PARTS_SHIFT);  // lane 0 has a row
        auto each = [&](auto f) {
#pragma unroll
            for (int c = 0; c < 4; ++c) total[0][c] = f(total[0][c], c);
        };
        if (parts_log2 > 0) each([&](float v, int c) { return v + other<1>(total[1][c]); });
        if (parts_log2 > 1) each([](float v, int) { return v + other<2>(v); });
        if (parts_log2 > 2) each([](float v, int) { return v + other<4>(v); });
        if (parts_log2 > 3) each([](float v, int) { return v + other<8>(v); });
        if (parts_log2 > 4) each([](float v, int) { return add_row(v); });
        if (parts_log2 > 5) each([](float v, int) { return add_half(v); });
        const uint32_t part = (uint32_t)lane & ((1u << parts_log2) - 1u);
        if (word != STRIP_NO_ROW && part < Q) {
            float *dst = args.C + (size_t)row * N + col0;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                if (q & ((1 << parts_log2) - 1)) continue;
                const uint32_t n = 4 * ((uint32_t)q ^ turn);
                if (col0 + n + 4 <= N) {
                    *reinterpret_cast<f32x4_unaligned *>(dst + n) = total[q];
                } else {
                    for (uint32_t c = 0; c < 4; ++c)
                        if (col0 + n + c < N) dst[n + c] = total[q][c];
                }
            }
        }
    }
}

// ---------------------------------------------------------------- builder
//
// The same units, order and bytes as the builder on the host makes (spmm_strips_build.h says why that order): the rows' entries
// band by band and class by class (class_kernel), then every unit in a band by a wave of its own, lane by lane what the host's
// loops do one after the other (order_kernel).  Plan and product in ms, each plan released before the next:
//                                    strips   built on the host   tiles of 16 rows   chunks
//   4096 x 4096, 80 %, 64 columns     0.79           5.7               0.87           10.1    (20 MB, of which the upload takes 0.5)
//   4096 x 4096, 95 %, 128 columns    0.55           2.2               0.65            3.0
// Working memory: 8 bytes an entry, 24 a row and 32 per row and band, and the units once more in bands; with 16 bytes an
// entry its allocation and release took 0.1 ms and 0.25 longer.

struct build_args {
    const int32_t *row_ptr;
    const float *vals;
    uint32_t *sorted;   // place in the band | number in the row << 16: the entries, a row's band by band and class by class
    uint32_t *classes;  // per row and band: entries; how many before its classes 1 .. 7
    uint32_t *flags;    // a word each for BAD_*, not zero where found
    uint32_t *units;
    uint32_t *rows;
    const uint32_t *order;  // the rows, longest first
    const u32x4 *list;      // the units
    char *stream;
    int64_t M;
    uint32_t nnz, places;  // units in a band
    int32_t K, bands, band_rows;
    builder::pull values;  // some of them, on their way beside the ordering
};
constexpr uint32_t NOTHING = ~0u;  // instead of an entry (its place is below the rows of a band)
constexpr int BAD_COLUMN = 0, BAD_ORDER = 1;

// One wave per row.
template <typename Col> __global__ __launch_bounds__(256) void class_kernel(const build_args args, const Col *col_idx)
{
    const int64_t row = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t lane = threadIdx.x & 63;
    if (row >= args.M) return;
    const int32_t first = args.row_ptr[row], end = args.row_ptr[row + 1];
    bool outside = false, disorder = false;
    for (int32_t band = 0, at = first; band < args.bands; ++band) {
        int32_t stop = end;
        if (band + 1 < args.bands) {  // the first entry beyond the band
            int32_t low = at;
            while (low < stop) {
                const int32_t middle = low + (stop - low) / 2;
                if ((int64_t)col_idx[middle] < (int64_t)(band + 1) * args.band_rows) low = middle + 1;
                else stop = middle;
            }
        }
        // Four loads at a time: one after the other they would take all of the kernel's time (25 us for the matrix above).
        constexpr int AHEAD = 4;
        int32_t c[AHEAD];
        auto load = [&](uint32_t q0, bool check) {
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) {
                const uint32_t q = q0 + 64u * k + lane;
                c[k] = q < (uint32_t)stop ? (int32_t)col_idx[q] : 0;
                if (check && q < (uint32_t)stop) {
                    outside |= (uint32_t)c[k] >= (uint32_t)args.K;
                    disorder |= q > (uint32_t)first && (int32_t)col_idx[q - 1] > c[k];
                }
            }
        };
        // the lanes whose column is of class x
        struct masks {
            uint64_t in, bit[3];
            __device__ uint64_t of(uint32_t x) const { return in & (x & 1 ? bit[0] : ~bit[0]) & (x & 2 ? bit[1] : ~bit[1]) & (x & 4 ? bit[2] : ~bit[2]); }
        };
        auto masks_of = [&](uint32_t q, int32_t column) {
            masks m;
            m.in = __ballot(q < (uint32_t)stop);
#pragma unroll
            for (int i = 0; i < 3; ++i) m.bit[i] = __ballot((column >> i & 1) != 0);
            return m;
        };
        const uint32_t mine = lane & 7;  // the class that the lane counts
        uint32_t n = 0;
        for (uint32_t q0 = (uint32_t)at; q0 < (uint32_t)stop; q0 += 64 * AHEAD) {
            load(q0, true);
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) n += (uint32_t)__popcll(masks_of(q0 + 64u * k + lane, c[k]).of(mine));
        }
        uint32_t before = n;  // and then, how many come before it
        for (uint32_t m = 1; m < 8; m *= 2) {
            const uint32_t less = (uint32_t)__shfl_up((int)before, m);
            if (mine >= m) before += less;
        }
        before -= n;
        if (lane < 8) args.classes[((size_t)row * (uint32_t)args.bands + (uint32_t)band) * 8 + lane] = lane == 0 ? (uint32_t)(stop - at) : before;
        for (uint32_t q0 = (uint32_t)at; q0 < (uint32_t)stop; q0 += 64 * AHEAD) {
            load(q0, false);
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) {
                const uint32_t q = q0 + 64u * k + lane;
                const masks m = masks_of(q, c[k]);
                const uint32_t to = (uint32_t)__shfl((int)before, c[k] & 7) + (uint32_t)__popcll(m.of((uint32_t)c[k] & 7u) & ((1ull << lane) - 1ull));
                if (q < (uint32_t)stop) args.sorted[(size_t)at + to] = ((uint32_t)(c[k] - band * args.band_rows) & 0xFFFFu) | (q - (uint32_t)first) << 16;
                before += (uint32_t)__popcll(m.of(mine));
            }
        }
        at = stop;
    }
    if (outside) args.flags[BAD_COLUMN] = 1;
    if (disorder) args.flags[BAD_ORDER] = 1;
}

// One wave per unit: the rows of its lanes, and its groups, in bands as many as its rows need there.
__global__ __launch_bounds__(64) void unit_kernel(const build_args args)
{
    const uint32_t unit = blockIdx.x, lane = threadIdx.x;
    const u32x4 u = args.list[unit];  // first row in the order, log2 of the parts, first group, groups
    const uint64_t at = (uint64_t)u[0] + (lane >> u[1]);
    const uint32_t row = at < (uint64_t)args.M ? args.order[at] : STRIP_NO_ROW;
    args.rows[(size_t)unit * 64 + lane] = row == STRIP_NO_ROW ? row : row | u[1] << STRIP_PARTS_SHIFT;
    uint32_t *to = args.units + (size_t)unit * (uint32_t)args.bands * 2;
    if (args.bands == 1) {
        if (lane < 2) to[lane] = lane == 0 ? u[2] : u[3];
        return;
    }
    for (int32_t band = 0; band < args.bands; ++band) {
        uint32_t n = 0;
        if (row != STRIP_NO_ROW) n = args.classes[((size_t)row * (uint32_t)args.bands + (uint32_t)band) * 8];
        uint32_t groups = (((n + (1u << u[1]) - 1u) >> u[1]) + STRIP_STEPS - 1) / STRIP_STEPS;
        for (int m = 1; m < 64; m *= 2) groups = max(groups, (uint32_t)__shfl_xor((int)groups, m));
        if (lane == 0) to[band * 2 + 1] = groups;
    }
}

// One workgroup: where the groups of every unit in a band begin; how many there are, and (behind) how many a unit has at most.
__global__ __launch_bounds__(1024) void begin_kernel(uint32_t *units, uint32_t n, uint32_t bands, uint64_t *total)
{
    __shared__ uint64_t sums[1024];
    __shared__ uint32_t longest;
    if (threadIdx.x == 0) longest = 0;
    const uint32_t share = (n + 1023) / 1024, first = min(n, threadIdx.x * share), end = min(n, first + share);
    uint64_t sum = 0;
    for (uint32_t k = first; k < end; ++k) sum += units[(size_t)k * 2 + 1];
    sums[threadIdx.x] = sum;
    __syncthreads();
    for (uint32_t m = 1; m < 1024; m *= 2) {
        const uint64_t more = threadIdx.x >= m ? sums[threadIdx.x - m] : 0;
        __syncthreads();
        sums[threadIdx.x] += more;
        __syncthreads();
    }
    uint64_t at = sums[threadIdx.x] - sum;
    for (uint32_t k = first; k < end; ++k) {
        units[(size_t)k * 2] = (uint32_t)at;
        at += units[(size_t)k * 2 + 1];
    }
    uint32_t most = 0;
    for (uint32_t k = threadIdx.x * bands; k < n; k += 1024 * bands) {
        uint32_t of_unit = 0;
        for (uint32_t b = 0; b < bands; ++b) of_unit += units[(size_t)(k + b) * 2 + 1];
        most = max(most, of_unit);
    }
    atomicMax(&longest, most);
    __syncthreads();
    if (threadIdx.x == 1023) {
        total[0] = sums[1023];
        total[1] = longest;
    }
}

// One wave per unit in a band.  Eight threads next to each other are the lanes that must not collide; what they propose goes
// around between them as a bit of a byte per turn.  Bound by the chain of a step's 300 instructions: 4096 x 4096, 80 %
// pruned, 104 steps, 78 us (with eight turns of one lane each and a shuffle 260).  It writes places and, where the values will
// be, the entries: so it needs no values, and the first workgroups copy a piece of those meanwhile (two of the three that the
// pinned memory holds would leave the next ones waiting).
__global__ __launch_bounds__(256) void order_kernel(const build_args args)
{
    const uint32_t pulling = args.values.n ? builder::PULL_BLOCKS : 0u;
    if (blockIdx.x < pulling) {
        builder::run_pull(args.values, blockIdx.x);
        return;
    }
    const uint32_t at_place = (blockIdx.x - pulling) * 4 + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (at_place >= args.places) return;
    const uint32_t unit = at_place / (uint32_t)args.bands, band = at_place % (uint32_t)args.bands;
    const uint32_t i = threadIdx.x & 7, set = threadIdx.x >> 3 & 7, j = 2 * i + (set & 1);
    const uint32_t lane = (set >> 2) * 32 + ((set & 2 ? 0x7421u : 0x6530u) >> (j / 4 * 4) & 15u) * 4 + j % 4;  // strip_lane(set / 2, i, set % 2)
    const uint32_t word = args.rows[(size_t)unit * 64 + lane], log2 = args.rows[(size_t)unit * 64] >> STRIP_PARTS_SHIFT, x = lane & ((1u << log2) - 1u);
    const uint32_t first = args.units[(size_t)at_place * 2], groups = args.units[(size_t)at_place * 2 + 1];
    uint32_t at[9] = {}, begin = 0;  // of the row's entries in the band: how many before a class; the first
    if (word != STRIP_NO_ROW) {
        const uint32_t row = word & ((1u << STRIP_PARTS_SHIFT) - 1u);
        const uint32_t *words = args.classes + (size_t)row * (uint32_t)args.bands * 8;
        begin = (uint32_t)args.row_ptr[row];
        for (uint32_t b = 0; b < band; ++b) begin += words[b * 8];
#pragma unroll
        for (int c = 1; c < 8; ++c) at[c] = words[band * 8 + c];
        at[8] = words[band * 8];
    }
    // the lane has those of them whose number modulo the row's parts is x
    auto mine = [&](uint32_t n) { return (int32_t)((n + (1u << log2) - 1u - x) >> log2); };
    int32_t next[8], count[8], most = 0;
    uint32_t has = 0, rich = 0, above = 0;
    auto sum_of_all = [](int32_t v) {  // over the eight
        v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, true);
        v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, true);
        return v + __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, true);
    };
    auto of_all = [](uint32_t v) {
        v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);
        v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true);
        return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);
    };
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        next[c] = mine(at[c]);
        count[c] = mine(at[c + 1]) - next[c];
        has |= (uint32_t)(count[c] > 0) << c;
        const int32_t sum = sum_of_all(count[c]);
        most = max(most, max(sum, __shfl_xor(sum, 8)));
    }
    int32_t left = mine(at[8]);
    const int32_t steps = (int32_t)(groups * STRIP_STEPS), extra = max(0, most - steps);
    int32_t part = 0;  // (t + 1) * extra modulo steps
    auto weigh = [&] {  // once a group
        const int32_t all = sum_of_all(left) / 8, own = left / 8;
        rich = above = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            rich |= (uint32_t)(count[c] > own) << c;
            above |= (uint32_t)(sum_of_all(count[c]) > all) << c;
        }
    };
    auto choose = [&](int32_t t) {  // place of the entry that the lane takes in step t
        bool twice = extra >= steps;
        if (!twice) {
            part += extra;
            twice = part >= steps;
            part -= twice ? steps : 0;
        }
        const uint32_t turn = (i - (uint32_t)t) & 7u, from = (i + (uint32_t)t) & 7u, shift = (turn & 3u) * 8u;
        const uint32_t before_low = turn < 4 ? (1u << shift) - 1u : ~0u, before_high = turn < 4 ? 0u : (1u << shift) - 1u;
        const bool waits = left < steps - t;
        uint32_t take = has >> from & 1u ? from : 8u;  // 8: none
        uint32_t once = of_all(take < 8 ? 1u << from : 0u), two = 0;
#pragma unroll
        for (int last = 0; last < 2; ++last) {
            const uint32_t can = has & ~(twice ? two : once);
            const bool idle = take < 8 || (can == 0 && (!last || waits));
            const uint32_t of = can ? can : has, both = of & rich & above, one = of & rich ? of & rich : of & above;
            const uint32_t best = both ? both : one ? one : of;
            const uint32_t choice = (uint32_t)__builtin_ctz(best << 8 | (best >> from << from) | 0x10000u) & 7u;
            const uint32_t bit = idle ? 0u : 1u << (choice + shift);
            const uint32_t low = of_all(turn < 4 ? bit : 0u), high = of_all(turn < 4 ? 0u : bit);  // a byte per turn
            auto fold = [](uint32_t l, uint32_t h, uint32_t &once, uint32_t &two) {               // classes in a byte, in two
                once = l | h;
                two = l & h;
                two |= two >> 16 | (once & once >> 16);
                once |= once >> 16;
                two = (two | two >> 8 | (once & once >> 8)) & 255u;
                once = (once | once >> 8) & 255u;
            };
            uint32_t earlier, earlier_two, all, all_two;
            fold(low & before_low, high & before_high, earlier, earlier_two);
            fold(low, high, all, all_two);
            const uint32_t full = twice ? two | (once & earlier) | earlier_two : once | earlier;
            if (!idle && (!(full >> choice & 1u) || (last && !waits))) take = choice;
            two |= (once & all) | all_two;
            once |= all;
        }
        uint32_t k = 0;
        const uint32_t bit = 1u << take;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int32_t is = (int32_t)(bit >> c & 1u);
            k = is ? (uint32_t)next[c] : k;
            next[c] += is;
            count[c] -= is;
            has &= ~((uint32_t)(count[c] == 0) << c);
        }
        left -= take < 8;
        return take < 8 ? begin + x + (k << log2) : NOTHING;
    };
    uint32_t taken[2][STRIP_STEPS];  // entries; written when the next group has been chosen
    char *out = args.stream + (size_t)first * STRIP_GROUP_BYTES;
    auto group = [&](uint32_t g, uint32_t (&e)[STRIP_STEPS]) {
        weigh();
#pragma unroll
        for (int k = 0; k < STRIP_STEPS; ++k) {
            const uint32_t from = choose((int32_t)(g * STRIP_STEPS) + k);
            e[k] = from == NOTHING ? NOTHING : args.sorted[from];
        }
    };
    auto store = [&](uint32_t g, const uint32_t (&e)[STRIP_STEPS]) {
        uint32_t place[STRIP_STEPS];
#pragma unroll
        for (int k = 0; k < STRIP_STEPS; ++k) place[k] = e[k] == NOTHING ? (uint32_t)args.band_rows : e[k] & 0xFFFFu;
        *reinterpret_cast<u32x4 *>(out + (size_t)g * STRIP_GROUP_BYTES + lane * 16) = u32x4{e[0], e[1], e[2], e[3]};
        *reinterpret_cast<u32x2 *>(out + (size_t)g * STRIP_GROUP_BYTES + 1024 + lane * 8) = u32x2{place[0] | place[1] << 16, place[2] | place[3] << 16};
    };
    if (groups == 0) return;
    group(0, taken[0]);
    uint32_t g = 1;
    for (; g + 1 < groups; g += 2) {
        group(g, taken[1]);
        store(g - 1, taken[0]);
        group(g + 1, taken[0]);
        store(g, taken[1]);
    }
    if (g < groups) {
        group(g, taken[1]);
        store(g - 1, taken[0]);
        store(g, taken[1]);
    } else {
        store(g - 1, taken[0]);
    }
}

// Eight waves per unit in a band: the values in place of the entries.
__global__ __launch_bounds__(512) void value_kernel(const build_args args)
{
    const uint32_t lane = threadIdx.x & 63, word = args.rows[(size_t)(blockIdx.x / (uint32_t)args.bands) * 64 + lane];
    const uint32_t first = args.units[(size_t)blockIdx.x * 2], groups = args.units[(size_t)blockIdx.x * 2 + 1];
    const float *vals = args.vals + (word == STRIP_NO_ROW ? 0 : args.row_ptr[word & ((1u << STRIP_PARTS_SHIFT) - 1u)]);
    char *at = args.stream + (size_t)first * STRIP_GROUP_BYTES + lane * 16;
    for (uint32_t g = threadIdx.x >> 6; g < groups; g += 8) {
        const u32x4 e = *reinterpret_cast<const u32x4 *>(at + (size_t)g * STRIP_GROUP_BYTES);
        f32x4 v;
#pragma unroll
        for (int k = 0; k < STRIP_STEPS; ++k) v[k] = e[k] == NOTHING ? 0.0f : vals[e[k] >> 16];
        *reinterpret_cast<f32x4 *>(at + (size_t)g * STRIP_GROUP_BYTES) = v;
    }
}

hipError_t build(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, int64_t N, strips::start &begun,
                 StripPlan &p, int &status)
{
    const int64_t nnz = row_ptr[M];
    hipError_t e;
#define TRY(x) do { e = (x); if (e != hipSuccess) return e; } while (0)
    builder::workshop memory;
    builder::uploader upload;  // (released before the memory)
    const bool staged = upload.begin(K, col_idx, vals, nnz, memory.stream), narrow = staged && upload.narrow_columns();
    strips::band_sizes(K, p);
    const int64_t bands = p.bands;
    // 256 threads per four rows; 32 bytes of working memory per row and band
    if (M > ((int64_t)1 << 26) - 8 || M * bands > (int64_t)1 << 26) { status = STRIPS_NOT_POSSIBLE; return hipSuccess; }
    // (a unit has a row at least; the columns, and when they have been read the values in their place)
    const size_t at_words = memory.reserve((size_t)M * 24 + 1024), at_entries = memory.reserve((size_t)nnz * 4);
    const size_t at_sorted = memory.reserve((size_t)nnz * 4), at_classes = memory.reserve((size_t)(M * bands) * 32);
    TRY(memory.take());
    const hipStream_t s = memory.stream;
    int32_t *d_col = memory.at<int32_t>(at_entries);
    uint32_t *d_words = memory.at<uint32_t>(at_words);
    uint64_t *answer = reinterpret_cast<uint64_t *>(d_words) + 2;  // behind four words of flags: groups, those of the longest unit
    const size_t front = ((size_t)M + 9 + 63) / 64 * 64, list = ((size_t)M + 3) / 4 * 4;
    build_args a{reinterpret_cast<const int32_t *>(d_words + 8), memory.at<float>(at_entries), memory.at<uint32_t>(at_sorted),
                 memory.at<uint32_t>(at_classes), staged ? upload.flags() : d_words, nullptr, nullptr, d_words + front,
                 reinterpret_cast<const u32x4 *>(d_words + front + list), nullptr, M, (uint32_t)nnz, 0, (int32_t)K, p.bands, p.band_rows, {}};
    // ---- while other threads fill the first pinned memory: the rows' order and the units
    strips::begin(M, K, row_ptr, N, begun);
    const std::vector<uint32_t> &order = begun.r.order;
    const std::vector<strips::unit> &units = begun.units;
    static_cast<StripSizes &>(p) = begun.sizes;
    const int64_t n_units = (int64_t)units.size(), places = n_units * bands;
    const size_t n_words = strips::unit_words(n_units, bands);
    const uint32_t longest = begun.r.length[0];
    // an entry's number in its row in 16 bits (so a unit has 2^14 groups in a band at most); blocks of 512 threads
    if (longest > 65535 || places >= (int64_t)1 << 23) { status = STRIPS_NOT_POSSIBLE; return hipSuccess; }
    // flags, groups, the row pointer; the order; the units in four words each (unit_kernel)
    std::vector<uint32_t> words(front + list + (size_t)n_units * 4, 0u);
    std::copy(row_ptr, row_ptr + M + 1, words.begin() + 8);
    std::copy(order.begin(), order.end(), words.begin() + (ptrdiff_t)front);
    uint64_t groups = 0;
    uint32_t *to = words.data() + front + list;
    for (const strips::unit &u : units) {
        const int64_t n = bands == 1 ? u.steps / STRIP_STEPS : 0;
        for (uint64_t w : {(uint64_t)u.first, (uint64_t)u.parts_log2, groups, (uint64_t)n}) *to++ = (uint32_t)w;
        groups += (uint64_t)n;
    }
    a.places = (uint32_t)places;
    TRY(upload.copy_words(words, d_words));
    if (staged) {
        TRY(upload.copy(0, reinterpret_cast<char *>(d_col)));
        if (upload.column_outside()) { status = 2; return hipSuccess; }
    } else {
        TRY(hipMemcpyWithStream(d_col, col_idx, (size_t)nnz * 4, hipMemcpyHostToDevice, s));
    }
    if (narrow) hipLaunchKernelGGL(class_kernel<uint16_t>, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, s, a, reinterpret_cast<const uint16_t *>(d_col));
    else hipLaunchKernelGGL(class_kernel<int32_t>, dim3((unsigned)((M + 3) / 4)), dim3(256), 0, s, a, d_col);
    TRY(hipGetLastError());
    TRY(upload.look());
    // the plan's memory, once it is known how much; in bands the units wait in memory of their own
    auto take_plan = [&]() -> hipError_t {
        if (groups >= (1ull << 32)) { status = STRIPS_NOT_POSSIBLE; return hipSuccess; }
        const hipError_t failed = hipMalloc(reinterpret_cast<void **>(&p.d_units), n_words * 4 + (size_t)groups * STRIP_GROUP_BYTES);
        if (failed != hipSuccess) return failed;
        a.units = p.d_units;
        p.d_stream = p.d_units + n_words;
        a.stream = reinterpret_cast<char *>(p.d_stream);
        return hipSuccess;
    };
    struct units_in_waiting {
        uint32_t *p = nullptr;
        hipStream_t s;
        ~units_in_waiting() { (void)give_back(); }
        hipError_t give_back()
        {
            uint32_t *const q = p;
            p = nullptr;
            return q ? hipFreeAsync(q, s) : hipSuccess;
        }
    } waiting;
    waiting.s = s;
    if (bands == 1) {
        TRY(take_plan());
        if (status) return hipSuccess;
    } else {
        TRY(hipMallocAsync(reinterpret_cast<void **>(&waiting.p), n_words * 4, s));
        a.units = waiting.p;
    }
    a.rows = a.units + places * 2;
    hipLaunchKernelGGL(unit_kernel, dim3((unsigned)n_units), dim3(64), 0, s, a);
    TRY(hipGetLastError());
    uint32_t got[8] = {};  // flags, groups, those of the longest unit
    auto refused = [&] {
        const uint32_t *flags = staged ? upload.flags() : got;
        status = flags[BAD_COLUMN] ? 2 : flags[BAD_ORDER] ? STRIPS_NOT_POSSIBLE : 0;
        return status != 0;
    };
    if (bands > 1) {
        hipLaunchKernelGGL(begin_kernel, dim3(1), dim3(1024), 0, s, a.units, (uint32_t)places, (uint32_t)bands, answer);
        TRY(hipGetLastError());
        TRY(hipMemcpyWithStream(got, d_words, sizeof got, hipMemcpyDeviceToHost, s));
        if (refused()) return hipSuccess;
        std::memcpy(&groups, got + 4, 8);
        p.steps = (int64_t)groups * STRIP_STEPS;
        p.longest = (int64_t)got[6] * STRIP_STEPS;
        begun.beaten = begun.others.faster_than_counted(p, K);
        if (begun.beaten) { status = STRIPS_NOT_POSSIBLE; return hipSuccess; }
        TRY(take_plan());
        if (status) return hipSuccess;
        TRY(hipMemcpyAsync(a.units, waiting.p, n_words * 4, hipMemcpyDeviceToDevice, s));
        a.rows = a.units + places * 2;
    }
    TRY(upload.next_values(memory.at<char>(at_entries), a.values));
    hipLaunchKernelGGL(order_kernel, dim3((unsigned)((places + 3) / 4) + (a.values.n ? builder::PULL_BLOCKS : 0u)), dim3(256), 0, s, a);
    TRY(hipGetLastError());
    TRY(upload.launched());
    if (staged) TRY(upload.copy(1, memory.at<char>(at_entries)));
    else TRY(hipMemcpyWithStream(d_col, vals, (size_t)nnz * 4, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(value_kernel, dim3((unsigned)places), dim3(512), 0, s, a);
    TRY(hipGetLastError());
    if (!staged) TRY(hipMemcpyWithStream(got, d_words, sizeof got, hipMemcpyDeviceToHost, s));
    TRY(waiting.give_back());
    TRY(memory.give_back());
    TRY(hipStreamSynchronize(s));
    if (refused()) return hipSuccess;
    upload.arrived();
#undef TRY
    p.n_units = n_units;
    p.steps = (int64_t)groups * STRIP_STEPS;
    strips::launches(p, K);
    p.device_bytes = (int64_t)((size_t)groups * STRIP_GROUP_BYTES + n_words * 4);
    p.built_on_device = true;
    builder::staging.count_plan(1);
    status = 0;
    return hipSuccess;
}

}  // namespace

// Strips of the first of two sets, or all.  In one set every XCD fetches all of B into its L2, one fourth of a line per strip,
// before its workgroups multiply, and an eighth of the entries; in two sets, one set's places before the other's, half of B and a quarter of the
// entries.  That pays where the entries are few beside B and the sets share no line.  us in one set and in two, plans and B in turn:
//   entries / B   0.7   1200 x 4800, 90 %, 256 columns   18.8 and 18.0     4096 x 4096, 97 %, 256 columns    16.7 and 15.9
//                 2     8192 x 8192, 98 %, 128           23.2 and 22.2     4096 x 8192, 97 %, 128            20.8 and 19.7
//                 2.6   4096 x 4096, 95 %, 128           12.9 and 12.4     4096 x 16384, 95 %, 128           43.7 and 42.1
//                 6     5000 x 4000, Zipf, 128           21.1 both
//                 11    8968 x 2473, 92 %, 96            14.0 and 14.2     4096 x 4096, 80 %, 64 (14)        16.4 and 16.6
// Rows that are not whole lines: 2 % slower to 1 % faster (110 to 250 columns).  Sets of 40 columns and fewer: up to 14 % slower.
// 39 random products that it takes 3.7 % faster on average, 2 % slower at worst; 21 others 0.98 to 1.06 times as fast in two sets, 1.01 on average.
uint32_t spmm_strips_of_set(int64_t steps, int64_t K, int32_t N)
{
    const int64_t strips = ((int64_t)N + STRIP_COLS - 1) / STRIP_COLS, half = ((strips + 1) / 2 + 3) / 4 * 4;  // (four strips: a line)
    const double entries = (double)steps * (STRIP_GROUP_BYTES / STRIP_STEPS), b = 4.0 * (double)K * (double)N;
    return (uint32_t)(N % 32 == 0 && strips >= 16 && entries < 8.0 * b ? half : strips);
}

int spmm_strips_execute(const StripPlan &p, int64_t K, const float *B, int32_t N, float *C, void *stream)
{
    const int64_t strips = ((int64_t)N + STRIP_COLS - 1) / STRIP_COLS;
    int64_t groups = 0;
    if (strips <= StripPlan::KNOWN) groups = p.groups[strips];
    else strip_time(p, K, N, &groups);
    strip_args a{reinterpret_cast<const char *>(p.d_stream), reinterpret_cast<const u32x2 *>(p.d_units), p.d_rows(), B, C, (uint64_t)K * (uint64_t)N * 4u, 0, 0,
                 (int32_t)K, N, p.bands, p.band_rows, (uint32_t)p.n_units, (uint32_t)groups, (uint32_t)strips, spmm_strips_of_set(p.steps, K, N), 0};
    a.n_places = a.n_groups * a.n_strips;
    const bool wide = (uint64_t)N * 4u * 32u >= (1ull << 32);
    const auto kernel = p.bands > 1 ? (wide ? spmm_strips_kernel<true, true> : spmm_strips_kernel<true, false>)
                                    : (wide ? spmm_strips_kernel<false, true> : spmm_strips_kernel<false, false>);
    // HIP refuses a grid of 2^32 threads or more
    const uint32_t most = (uint32_t)(((1ull << 32) - 1) / (64 * STRIP_WAVES) / 8 * 8);
    for (uint32_t first = 0; first < a.n_places; first += most) {
        a.first = first;
        a.share = (std::min(a.n_places - first, most) + 7) / 8;
        const unsigned blocks = a.share * 8u;
        const hipError_t e = launch_kernel(kernel, dim3(blocks), 64 * STRIP_WAVES, (unsigned)(p.band_rows + 1) * STRIP_ROW_BYTES, (hipStream_t)stream, a);
        if (e != hipSuccess) return (int)e;
    }
    return (int)hipSuccess;
}

int spmm_strips_build_on_device(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, int64_t N,
                                strips::start &begun, StripPlan &out)
{
    out = StripPlan();
    int status = 0;
    const hipError_t e = build(M, K, row_ptr, col_idx, vals, N, begun, out, status);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        status = e == hipErrorOutOfMemory ? 3 : 4;
    }
    if (status != 0) spmm_strips_release(out);
    return status;
}

void spmm_strips_release(StripPlan &p)
{
    if (p.d_units) (void)hipFree(p.d_units);
    if (p.built_on_device) builder::staging.count_plan(-1);
    p = StripPlan();
}
