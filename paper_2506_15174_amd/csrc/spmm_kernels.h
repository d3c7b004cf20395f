// Host-side launch interface of the gfx950 kernels (internal; the public C ABI
// is include/spmm.h).
#ifndef SPMM_KERNELS_H
#define SPMM_KERNELS_H

#include <stddef.h>
#include <stdint.h>

#include "spmm_format.h"
#include "spmm_places.h"

// Waves per SIMD an instance is compiled for (its register budget: 512 / waves).  Measured on
// the pruned-layer shapes with every depth forced: past two or three chunks in flight a deeper
// pipeline buys nothing (the memory path, not the number of requests a wave has outstanding,
// paces the gather), while every further resident wave hides more of the chunk's dependent
// chain (header, row branches, value reads).  So each instance takes the shallowest pipeline
// that keeps the loads flowing and the occupancy its tile allows: eight-row tiles, 32 registers by themselves, 4 waves
// (6 on four slices; on eight, sized for 6, 68 registers spilled and it ran 10-28 % slower), four-row tiles 4 waves on two slices and 8 otherwise, shorter tiles 6 to
// 8.  Wider chunks (UFKT > 8) give a slice two column slots per chunk: 8 waves (6 with eight
// rows) on 16 columns, where 6 (4) are as fast but for the blocks that may be dealt (workgroups_per_unit; single rows at 18 to 32 columns, in
// us: 2048 x 4096, 90 % lognormal, 8.6 -> 8.0, 11461 x 2261, 95 %, 11.4 -> 11.2, ten others within 1.5 %); windows of 2048 words (UFKT >= 32) cap a compute unit at two workgroups.
// Every budget is one the instance fits without spilling (the build checks it): a spilled
// register could be the destination of a B row still in flight.  64-bit addressing costs a
// register more per column slot, so those instances get the budget of two waves fewer.
constexpr int waves_per_simd(int S, int UFI, int UFKT, bool WIDE)
{
    const int narrow = UFKT >= 32  ? 4
                       : UFKT == 16 ? (UFI > 4 ? 6 : 8)
                       : S == 1     ? 4
                       : UFI == 8   ? (S == 2 ? 4 : 6)
                       : UFI == 4   ? (S == 2 ? 4 : 8)
                       : UFI == 2   ? (S == 2 ? 6 : 8)
                                    : 8;
    return WIDE ? (narrow > 4 ? narrow - 2 : 2) : narrow;
}

// Chunks of B rows that a wave of an instance has in flight: the shallowest pipeline that keeps the
// loads flowing (see waves_per_simd); one column slot per slice (8 slices) needs more chunks
// in flight for the same number of requests.  Single rows in two slices make four loads per chunk, and
// up to 32 waves per compute unit keep the gather busy by themselves: looking a chunk ahead only costs work at
// the ends of the short windows (4096 x 4096, 95 % pruned, 128 columns: 18.0 us with two in flight, 17.4 with
// one; 22 even and uneven matrices 2 to 12 % faster).  64-bit addresses keep two, and so does a caller who asks for more.
// Plans made for narrow B, two: a wave has five to thirty of their wide chunks, and every further one in flight lengthens the start of
// its window (8192 x 8192, 98 % pruned, 32 columns: 9.5 us with four, 9.0 with three, 8.6 with two; 40 of
// 48 plans of one to eight rows are fastest with two or, by less than 2 %, three).
constexpr int chunk_depth(int UFI, int UFKT, int S)
{
    return UFKT > spmm_fmt::UFK ? 2
           : S == 1             ? 3
           : S == 2             ? (UFI == 1 ? 1 : 2)
           : S == 4             ? (UFI >= 4 ? 3 : 2)
           : UFI >= 4           ? 4
           : UFI == 2           ? 6
                                : 8;
}

// Workgroups of an instance that share a compute unit: by its registers, and by 160 KiB of LDS.
constexpr int workgroups_per_unit(int S, int UFI, int UFKT, bool WIDE)
{
    const int by_waves = waves_per_simd(S, UFI, UFKT, WIDE) * 4 / spmm_fmt::WAVES_PER_WG;
    const int by_lds = 160 * 1024 / (spmm_fmt::WAVES_PER_WG * spmm_fmt::win_words(UFKT) * 4);
    return by_waves < by_lds ? by_waves : by_lds;
}

struct spmm_launch_args {
    const uint32_t *stream; // DEVICE staging windows: headers, column indices, value bits
    const uint32_t *wins;   // DEVICE window table
    const uint32_t *items;  // DEVICE wave-slot descriptors, 16 per block
    const uint32_t *rowmap = nullptr; // DEVICE row of C per row of the plan, or null (same rows)
    int32_t n_blocks;       // workgroups to launch
    // The same descriptors in the order in which compute units are loaded evenly, idle blocks among them (deal_blocks), for a
    // launch of one column tile.  None: 0.
    const uint32_t *dealt = nullptr;
    int32_t n_dealt = 0;
    const float *B;         // DEVICE first column of the launch's first column tile
    uint32_t b_bytes;       // bytes of B reachable from that pointer (narrow addressing only)
    float *C;               // DEVICE first column of the launch's first column tile (of the slices' buffer when k_slices > 1)
    int32_t ldn;            // leading dimension of B (= N)
    int32_t ldc;            // leading dimension of what C points to
    int32_t width;          // columns of this launch: n_tiles tiles of tile_cols, the last maybe narrower
    int32_t tile_cols;      // columns per tile
    int32_t n_tiles;        // column tiles of this launch (grid y)
    uint32_t col_mask;      // bits of a column word that hold the column index
    uint32_t lds_pad = 0;   // extra LDS bytes per workgroup (never touched): caps the workgroups per CU
    int32_t heavy = 0;      // the plan's first blocks that are heavier than most (front_blocks)
    bool probe = false;     // launch the loads-only instance (32-bit addressing, tuned depth, chunks of 8 or 16)
    // Panels cut across workgroups (plans with n_cross > 0; else unused):
    float *cross_sums = nullptr;          // DEVICE n_tiles x n_cross_slots slots of ufi x 128 floats (scratch)
    const uint32_t *cross_table = nullptr;// DEVICE one entry per such panel: slots and rows of C
    uint32_t n_cross_slots = 0;
    int32_t n_cross = 0;
    // Plans cut along K (k_slices > 1; else unused): C above is the slices' buffer (k_slices x
    // slice_rows rows of ldc floats); a last launch adds the slices of the first M rows into C_out.
    int32_t k_slices = 1;
    int64_t slice_rows = 0, M = 0;
    float *C_out = nullptr;  // DEVICE first column of this launch in the caller's C
    int32_t ldc_out = 0;     // its leading dimension (= N)
};

// What a workgroup of a launch computes: the plan's block and the column tile.  Workgroups start in the order of x, then y.
// The first `front` blocks of all tiles come first, block by block, then the others tile by tile.
struct place {
    uint32_t block, tile;
};
// A launch and a workgroup of it for place_of on the host; a kernel hands over its arguments and blockIdx.
struct launch_shape {
    uint32_t n_blocks, n_tiles, front;
};
struct launch_group {
    uint32_t x, y;
};
template <typename args_t, typename at_t> SPMM_DEVICE place place_of(const args_t &args, const at_t &group)
{
    if (__builtin_expect(args.front == 0, 1)) return place{group.x, group.y};  // (one tile: without a taken branch)
    const uint32_t at = group.y * args.n_blocks + group.x, front = args.front * args.n_tiles;
    if (at < front) {
        const uint32_t block = at / args.n_tiles;
        return place{block, at - block * args.n_tiles};
    }
    const uint32_t rest = args.n_blocks - args.front, tile = (at - front) / rest;
    return place{args.front + at - front - tile * rest, tile};
}
// Two, four and eight tiles of 64 or 128 columns: all blocks.  Workgroups go to the eight XCDs in turn, so that an
// XCD's L2 sees the rows of one tile and fetches a half (a quarter, an eighth) of B, and the launch ends with the
// lightest blocks of all tiles.  48 even and uneven matrices at 256 columns: 10 % faster on average, at worst 5 % slower; 24 at 512: 14 and 4 %.  4096 x 4096, 5 %
// even, 256 columns 31.8 -> 29.5 us.  Not where the last tile is less
// than seven eighths of the others: its XCDs would be done early (even matrices at 200 columns 5 % slower on average, up to 10 %).
//
// Other launches of uneven plans: taken tile by tile, the heaviest blocks of the second tile start when the first has
// none left to hide them behind.  One block per compute unit comes first, of more or narrower tiles only those that are
// heavier than most: 1024 x 4096, 6 % in Zipf rows, 200 columns 33.9 -> 21.0 us; 1024 x 4096, 10 % lognormal, 25.1 -> 21.5.  The 48 at
// 200 and 224 columns: 4 and 5 % faster on average, at 384 2 %; Zipf rows gain most and some of them lose (16384 x 2048, 3 % kept, 12 % at 200 columns,
// 7 % at 384; 3000 x 4096, 5 % kept, 10 %).  Only the heavier blocks first at all widths: 2 % slower on average at 161 to 224 columns, 23 % at
// worst.  Tiles of 16 columns and less, which share the cache lines of B: none.
inline uint32_t front_blocks(const spmm_launch_args &a)
{
    const int32_t T = a.n_tiles, last = a.width - (T - 1) * a.tile_cols;
    if (T == 1 || a.tile_cols < 32) return 0;
    if ((T == 2 || T == 4 || T == 8) && a.tile_cols >= 64 && 8 * last >= 7 * a.tile_cols) return (uint32_t)a.n_blocks;
    const int32_t wanted = a.heavy > 0 && (a.tile_cols == 64 || (a.tile_cols > 64 && T == 2)) ? a.n_blocks : a.heavy;
    return (uint32_t)(wanted < 256 / T ? wanted : 256 / T);
}

// Enqueues one launch of n_tiles column tiles (plus the small launches that add the sums of
// panels cut across workgroups and of plans cut along K).  ufi = rows per panel of the plan (1, 2, 4, 8).
// slices = 2 / 4 / 8: four columns per lane (16-byte loads and stores at 4-byte alignment;
// the last lane of a tile may own fewer than four columns), tile of up to 128 / 64 / 32
// columns; slices = 1: one column per lane, tile of up to 64 columns.  wide = 64-bit
// addressing of B.  depth = chunks of B rows in flight (0 or anything deeper than the
// instance's tuned depth = the tuned depth).  Returns the hipError_t of the launch as int.
// ufk = columns per chunk of the plan: 8, or 16 / 32 / 64 with slices = 8 / 16 / 32 or 64 (tiles
// of 32 / 16 / 8 or 4 columns; 32-bit addressing and the tuned depth only).
int spmm_launch_chunks(const spmm_launch_args &a, int ufi, int ufk, int slices, bool wide, int depth, void *stream);

// The tuned depth of such a launch, for the tests (chunk_depth).
extern "C" int spmm_chunk_depth(int ufi, int ufk, int slices);

// Size of the library's statically allocated device scratch (one copy per device, held
// until the process ends).
#define SPMM_STATIC_SCRATCH_BYTES ((size_t)6 << 20)

// The current device's copy of that scratch: *ptr = its device address, *bytes = its size.
// The first call on a device asks the runtime for the address (no allocation: the array is
// part of the loaded code object); later calls return the kept value.  Returns a hipError_t.
int spmm_static_scratch(float **ptr, size_t *bytes);

#endif
