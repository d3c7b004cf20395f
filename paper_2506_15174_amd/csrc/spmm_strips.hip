// gfx950 executor of the strips path: C <- A x B with eight columns of B in LDS at a time (format: spmm_strips.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "spmm_strips.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
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

// v + v of another lane of the row of 16 (CTRL: a DPP permutation)
template <int CTRL> __device__ __forceinline__ float add_other(float v)
{
    return v + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, true));
}
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
// What bounds it: LDS (two reads of 4.3 cycles per step and wave, 1.2 times that with the collisions that the
// builder's order leaves) and the vector ALUs (8 multiply-adds and 3 others per step) about equally, 11 of the 17 cycles that a step takes, and
// before them the copy of the strip: the vector L1 fetches a line of 128 bytes for 32, 2 cycles, so 4096 rows take 3.6 us.
// Three plans in turn, on chunks and on strips: 4096 x 4096, 95 % pruned, 128 columns 17.4 and 14.3 us, 3001 x 2511, 85 % in lognormal
// rows, 200 columns 37.4 and 20.8.  Back to back 8968 x 2473, 92 %, 96 columns 37 and 14, 2432 x 6741, 91 %, 112 columns 37 and 19.
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
    const uint32_t N = (uint32_t)args.N, col0 = strip * STRIP_COLS, band_rows = (uint32_t)args.band_rows;
    const uint32_t half = (uint32_t)(lane & 1) * 16u;  // of its rows of the strip, which the lane reads first
    const int bands = BANDS ? args.bands : 1;

    if (threadIdx.x < 2) *reinterpret_cast<f32x4 *>(lds + band_rows * STRIP_ROW_BYTES + threadIdx.x * 16) = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    auto copy_band = [&](uint32_t band) {
        const uint32_t row0 = band * band_rows, rows = min(band_rows, (uint32_t)args.K - row0);
        if constexpr (WIDE) {
            for (uint32_t t = threadIdx.x; t < rows * 2; t += 64 * STRIP_WAVES) {
                const float *p = args.B + (uint64_t)(row0 + t / 2) * N;
                const uint32_t n = col0 + t % 2 * 4;
                f32x4 x;
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) x[c] = n + c < N ? p[n + c] : 0.0f;
                *reinterpret_cast<f32x4 *>(lds + t * 16) = x;
            }
        } else {
            // 32 rows at a time, two lanes a row.  (Past the end of B zeros, past the end of a row what follows: columns that C does not have.)
            const uint32_t off = (uint32_t)(lane / 2) * N * 4u + (uint32_t)(lane % 2) * 16u;
            for (uint32_t op = (uint32_t)wave; op * 32 < rows; op += STRIP_WAVES) {
                const uint64_t skip = ((uint64_t)(row0 + op * 32) * N + col0) * 4u, left = args.b_bytes - skip;
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
        f32x4 acc[STRIP_STEPS][2], total[2] = {};  // of the last groups; of all before them
        auto collect = [&] {
#pragma unroll
            for (int q = 0; q < 2; ++q) total[q] += (acc[0][q] + acc[1][q]) + (acc[2][q] + acc[3][q]);
#pragma unroll
            for (int e = 0; e < STRIP_STEPS; ++e) acc[e][0] = acc[e][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        };
#pragma unroll
        for (int e = 0; e < STRIP_STEPS; ++e) acc[e][0] = acc[e][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
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
            f32x4 x[2][2][2];  // rows of the strip: two steps each, read while the other two are multiplied
            auto read = [&](int k, int h) {
                const uint32_t two = places[k][h];
                uint32_t at[2];
                asm("v_mad_u32_u16 %0, %1, 32, %2" : "=v"(at[0]) : "v"(two), "v"(half));
                asm("v_mad_u32_u16 %0, %1, 32, %2 op_sel:[1,0,0,0]" : "=v"(at[1]) : "v"(two), "v"(half));
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    x[h][e][0] = *reinterpret_cast<const f32x4 *>(lds + at[e]);
                    x[h][e][1] = *reinterpret_cast<const f32x4 *>(lds + (at[e] ^ 16u));
                }
            };
            auto multiply = [&](int k, int h) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            acc[2 * h + e][q][c] = __builtin_fmaf(values[k][2 * h + e], x[h][e][q][c], acc[2 * h + e][q][c]);
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
                }
                if (g % 12 == 9) collect();
            }
        }
        if (!any) break;
        collect();
        // ---- the sums of the four steps, of the parts of a row; two lanes of a row store four columns each
        const bool odd = (lane & 1) != 0;
        f32x4 sum[2] = {odd ? total[1] : total[0], odd ? total[0] : total[1]};  // columns 0 .. 3 and 4 .. 7
        const uint32_t word = args.rows[(size_t)unit * 64u + (uint32_t)lane], row = word & ((1u << STRIP_PARTS_SHIFT) - 1u);
        const uint32_t parts_log2 = __builtin_amdgcn_readfirstlane(word >> STRIP_PARTS_SHIFT);  // lane 0 has a row
        auto all = [&](auto f) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c) sum[q][c] = f(sum[q][c]);
        };
        // (each pair of lanes has equal sums after the first step, each four after the second: mirrored lanes serve)
        if (parts_log2 > 0) all([](float v) { return add_other<0xB1>(v); });   // lanes 1 0 3 2
        if (parts_log2 > 1) all([](float v) { return add_other<0x4E>(v); });   // lanes 2 3 0 1
        if (parts_log2 > 2) all([](float v) { return add_other<0x141>(v); });  // the other four of eight
        if (parts_log2 > 3) all([](float v) { return add_other<0x140>(v); });  // the other eight of 16
        if (parts_log2 > 4) all([](float v) { return add_row(v); });
        if (parts_log2 > 5) all([](float v) { return add_half(v); });
        const uint32_t part = (uint32_t)lane & ((1u << parts_log2) - 1u);
        if (word != STRIP_NO_ROW && part < 2) {
            float *dst = args.C + (size_t)row * N + col0;
#pragma unroll
            for (uint32_t q = 0; q < 2; ++q) {
                if (parts_log2 > 0 && part != q) continue;
                if (col0 + 4 * q + 4 <= N) {
                    *reinterpret_cast<f32x4_unaligned *>(dst + 4 * q) = sum[q];
                } else {
                    for (uint32_t c = 0; c < 4; ++c)
                        if (col0 + 4 * q + c < N) dst[4 * q + c] = sum[q][c];
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
