// gfx950 executor of the strips path: C <- A x B with eight columns of B in LDS at a time (format: spmm_strips.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "spmm_strips.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
typedef float f32x4_unaligned __attribute__((ext_vector_type(4), aligned(4)));

struct strip_args {
    const char *stream;
    const u32x2 *units;
    const uint32_t *rows;
    const float *B;
    float *C;
    uint64_t b_bytes;   // bytes of B
    uint64_t n_places;  // strips of all groups
    uint64_t first;     // the launch's first
    int32_t K, N, bands, band_rows;
    uint32_t n_units, n_groups, n_strips;
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
// Why: a gather of rows of B from the vector L1 moves 64 bytes per cycle and compute unit at most (16 cycles per wave load), reads of LDS 256 where the
// lanes' banks differ; and a lane that owns a part of a row adds up by itself, without a cross-lane step per entry.  A lane holds
// four sums per column, for the four steps of a group: chains of a quarter of its entries.
//
// Every 12 groups they go to a total (8192 x 8192, 50 % kept: error against 64 bits 4.1e-7 without, 1.9e-7 with a total every 6).
//
// What bounds it: LDS (two reads of 4.3 cycles per step and wave, 1.15 times that with the collisions that the builder's order
// leaves), the vector ALUs (8 multiply-adds and 2 others per step) and the fetch of the entries (384 bytes per step) take about ten
// cycles each of the 15 that a step and wave takes of a compute unit; and before them the copy of the strip: the vector L1
// fetches a line of 128 bytes for 32, 2 cycles, so 4096 rows take 3.6 us.
// Three plans in turn, on chunks and on strips: 4096 x 4096, 95 % pruned, 128 columns 17.4 and 13.0 us, 3001 x 2511, 85 % in lognormal
// rows, 200 columns 37.4 and 17.4.  Back to back 8968 x 2473, 92 %, 96 columns 39 and 14.
//
// An accumulator's registers hold columns 1 0 3 2 of its four: a v_fmac of three registers that are all even or all odd takes 4.9
// cycles, else 2.8, and those of LDS hold them in order (1 to 3 % of the product).
template <bool BANDS, bool WIDE> __global__ __launch_bounds__(64 * STRIP_WAVES, STRIP_WAVES / 4) void spmm_strips_kernel(const strip_args args)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // Workgroups are dealt to the eight XCDs in turn: each takes an eighth of the places, next to each other, so that the strips of
    // a group, which read the same entries, share an L2.
    const uint64_t place = args.first + blockIdx.x % 8u * (gridDim.x / 8u) + blockIdx.x / 8u;
    if (place >= args.n_places) return;
    const uint32_t group = (uint32_t)(place / args.n_strips), strip = (uint32_t)(place % args.n_strips);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    constexpr int Q = STRIP_COLS / 4;  // fours of columns; the lane reads four i ^ turn of its rows as the i-th
    const uint32_t turn = (uint32_t)lane % Q, N = (uint32_t)args.N, col0 = strip * STRIP_COLS, band_rows = (uint32_t)args.band_rows;
    const int bands = BANDS ? args.bands : 1;

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
            // 1024 bytes at a time, Q lanes a row.  (Past the end of B zeros, past the end of a row what follows: columns that C does not have.)
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
    copy_band(0);
    bool copied = false;  // the first band, and waited for

    for (uint32_t unit = group + (uint32_t)wave * args.n_groups;; unit += STRIP_WAVES * args.n_groups) {
        const bool any = unit < args.n_units;
        if (!any && copied) break;
        f32x4 acc[STRIP_STEPS][Q], total[Q] = {};  // of the last groups; of all before them
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
            const u32x2 d = any ? args.units[(size_t)unit * (uint32_t)bands + (uint32_t)band] : u32x2{0u, 0u};
            const uint32_t first = __builtin_amdgcn_readfirstlane(d[0]), groups = __builtin_amdgcn_readfirstlane(d[1]);
            const char *stream = args.stream + (size_t)first * STRIP_GROUP_BYTES;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(stream), (short)0, (int)(groups * STRIP_GROUP_BYTES), 0x00020000);
            f32x4 values[3];  // of the group at work and the next two
            u32x2 places[3];
            auto fetch = [&](int k, uint32_t g) {  // nothing past the unit
                values[k] = __builtin_bit_cast(f32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, (int)(g * STRIP_GROUP_BYTES), 0));
                places[k] = __builtin_amdgcn_raw_buffer_load_b64(r, 1024 + lane * 8, (int)(g * STRIP_GROUP_BYTES), 0);
            };
            fetch(0, 0);
            fetch(1, 1);
            if (BANDS && band > 0) {
                __syncthreads();
                copy_band((uint32_t)band);
            }
            if (BANDS || !copied) __syncthreads();
            copied = true;
            f32x4 x[2][2][Q];  // rows of the strip: two steps each, read while the other two are multiplied
            auto read = [&](int k, int h) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    // (as an integer: the address of lds is 0, and to it the compiler would add)
                    uint32_t at;
                    if (e == 0) asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(places[k][h]), "n"(STRIP_ROW_BYTES), "v"(turn * 16u));
                    else asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(at) : "v"(places[k][h]), "n"(STRIP_ROW_BYTES), "v"(turn * 16u));
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
            // The compiler would move the loads to their first use.
            auto keep_order = [] { __builtin_amdgcn_sched_barrier(0); };
            read(0, 0);
            for (uint32_t g = 0; g < groups; g += 3) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (k > 0 && g + (uint32_t)k >= groups) break;
                    fetch((k + 2) % 3, g + (uint32_t)k + 2u);
                    keep_order();
                    read(k, 1);
                    keep_order();
                    multiply(k, 0);
                    keep_order();
                    read((k + 1) % 3, 0);
                    keep_order();
                    multiply(k, 1);
                    keep_order();
                }
                // (four registers in a row, not any four)
#pragma unroll
                for (int e = 0; e < STRIP_STEPS; ++e)
#pragma unroll
                    for (int q = 0; q < Q; ++q) asm volatile("" : "+v"(acc[e][q]));
                if (g % 12 == 9) collect();
            }
        }
        if (!any) break;
        collect();
        // ---- the sums of the parts of a row: lanes l and l ^ 1, then l and l ^ 2, each keep the fours that they read first (the other
        // one has four i of the lane as i ^ 1, i ^ 2); from then on a lane has one four
#pragma unroll
        for (int q = 0; q < Q; ++q) total[q] = __builtin_shufflevector(total[q], total[q], 1, 0, 3, 2);
        const uint32_t word = args.rows[(size_t)unit * 64u + (uint32_t)lane], row = word & ((1u << STRIP_PARTS_SHIFT) - 1u);
        const uint32_t parts_log2 = __builtin_amdgcn_readfirstlane(word >> STRIP_PARTS_SHIFT);  // lane 0 has a row
        auto each = [&](int q, auto f) {
#pragma unroll
            for (int c = 0; c < 4; ++c) total[q][c] = f(total[q][c], c);
        };
        if (parts_log2 > 0) {
#pragma unroll
            for (int q = 0; q < Q; q += 2) each(q, [&](float v, int c) { return v + other<1>(total[q + 1][c]); });
        }
        if (parts_log2 > 1) each(0, [&](float v, int c) { return v + other<2>(total[Q > 2 ? 2 : 0][c]); });
        if (parts_log2 > 2) each(0, [](float v, int) { return v + other<4>(v); });
        if (parts_log2 > 3) each(0, [](float v, int) { return v + other<8>(v); });
        if (parts_log2 > 4) each(0, [](float v, int) { return add_row(v); });
        if (parts_log2 > 5) each(0, [](float v, int) { return add_half(v); });
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

}  // namespace

int spmm_strips_execute(const StripPlan &p, int64_t K, const float *B, int32_t N, float *C, void *stream)
{
    const int64_t strips = ((int64_t)N + STRIP_COLS - 1) / STRIP_COLS;
    int64_t groups = 0;
    if (strips <= StripPlan::KNOWN) groups = p.groups[strips];
    else strip_time(p, K, N, &groups);
    strip_args a{reinterpret_cast<const char *>(p.d_stream), reinterpret_cast<const u32x2 *>(p.d_units), p.d_rows, B, C, (uint64_t)K * (uint64_t)N * 4u, 0, 0,
                 (int32_t)K, N, p.bands, p.band_rows, (uint32_t)p.n_units, (uint32_t)groups, (uint32_t)strips};
    a.n_places = (uint64_t)a.n_groups * a.n_strips;
    const bool wide = (uint64_t)N * 4u * 32u >= (1ull << 32);
    const auto kernel = p.bands > 1 ? (wide ? spmm_strips_kernel<true, true> : spmm_strips_kernel<true, false>)
                                    : (wide ? spmm_strips_kernel<false, true> : spmm_strips_kernel<false, false>);
    // HIP refuses a grid of 2^32 threads or more
    const uint64_t most = ((1ull << 32) - 1) / (64 * STRIP_WAVES) / 8 * 8;
    for (uint64_t first = 0; first < a.n_places; first += most) {
        a.first = first;
        const unsigned blocks = (unsigned)((std::min(a.n_places - first, most) + 7) / 8) * 8u;
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * STRIP_WAVES), (unsigned)(p.band_rows + 1) * STRIP_ROW_BYTES, (hipStream_t)stream, a);
    }
    return (int)hipGetLastError();
}
