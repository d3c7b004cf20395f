// Matrix-core path (internal): A in tiles, multiplied by MFMA instructions (fp32, or bf16 on values in three parts).
#ifndef SPMM_TILES_H
#define SPMM_TILES_H

#include <stddef.h>
#include <stdint.h>

// Format.  The rows are taken in panels of `rows` = R (32, 16 or 8) consecutive rows of A, the
// columns in steps of 16 * 64 / R columns.  The wave that multiplies a (panel, step) pair, a *block*,
// gives it to 16 matrix operands t of one element per lane l:
//   R = 32, 16   row l % R of the panel, column t * 64 / R + l / R of the step
//   R = 8        row t % 2 * 4 + l % 4, column t / 2 * 16 + l / 4
// A block stores
//   values     its entries, filled up to a multiple of eight with zeros; their order spreads the places of
//              the entries that a wave writes together over the banks of LDS
//   places     16 bits per entry: where the value goes in the expanded block, in bytes:
//              TILE_PLACE0 + ((t / 4 * 64 + l) * 4 + t % 4) * 4, or 0 for a filler
// Blocks lie panel by panel, step by step.
// offsets[panel * (n_steps + 1) + s] = start of block s of the panel in units of eight entries.
struct TilePlan {
    int32_t rows = 0;               // R; 0 = the plan holds no tiles
    int64_t n_panels = 0, n_steps = 0;
    int32_t loads = 4;              // runs of 256 entries the longest block has
    uint32_t *d_stream = nullptr;   // DEVICE blocks
    uint32_t *d_offsets = nullptr;  // DEVICE n_panels * (n_steps + 1) block starts
    int64_t stream_words = 0, device_bytes = 0;
    bool built = false;             // whole
    bool exact_parts = false;       // R = 32: every value is the sum of three bf16 numbers
    float largest = 0.0f;           // R = 32: size of the largest value
};

constexpr int TILE_OPERANDS = 16;
constexpr int TILE_PLACE0 = 16;

// Builds the tiles of A on the current device from host CSR arrays whose row pointer has been
// checked; the columns are checked here.  Status codes follow spmm_status_t; TILES_NOT_POSSIBLE:
// A cannot be stored this way (a column occurs twice in a row, more than 2^34 words of blocks, or
// 2^26 rows or blocks and more: the builder's launches).
constexpr int TILES_NOT_POSSIBLE = -1;
int spmm_tiles_build(int64_t M, int64_t K, const int32_t *row_ptr, const int32_t *col_idx, const float *vals, int32_t rows,
                     TilePlan &out);
void spmm_tiles_release(TilePlan &p);

// Estimated time of a product in us with panels of `rows` rows, and the column groups NB of a tile
// (1, 2 or 4) it runs with.  density = share of the entries kept, peak = the largest such share of a panel.
extern "C" double spmm_tiles_time(int rows, int64_t M, int64_t K, int64_t N, double density, double peak, int *NB);

// Column tiles of the first of the two sets in which those of panels of 16 rows come, half of the XCDs fetching each; all:
// one set.  stream_words: of the plan.
extern "C" uint32_t spmm_tiles_of_set(int rows, int64_t M, int64_t K, int32_t N, int64_t stream_words);

// Enqueues C <- A x B.  Returns the hipError_t of the launch as int.
int spmm_tiles_execute(const TilePlan &p, int64_t M, int64_t K, const float *B, int32_t N, float *C, void *stream);

#endif
