// Which widths a chunk plan's products run as two column tiles (spared_by_two_tiles in spmm_api.cpp), as spmm_execute hands them to the
// launcher, on the stand-ins of host_sources_on_stand_ins.cpp.
#define main main_of_host_sources
#include "host_sources_on_stand_ins.cpp"
#undef main

extern "C" int32_t spmm_chunk_tiles(const spmm_plan_t *plan, int32_t N, int32_t *tile_cols);

static std::vector<spmm_launch_args> on_columns(const spmm_plan_t *p, int N)
{
    static float word;  // B and C are only passed on
    launched.clear();
    REQUIRE(spmm_execute(p, &word, N, &word, nullptr) == SPMM_OK && !launched.empty());
    int32_t tile_cols = 0;
    REQUIRE(spmm_chunk_tiles(p, N, &tile_cols) == launched[0].n_tiles && tile_cols == launched[0].tile_cols);
    return launched;
}

// Chunks, and eight per block, on the fullest of 256 compute units that get the workgroups of a launch in turn, per column tile.
static int64_t fullest(const spmm_launch_args &l)
{
    const bool dealt = l.n_dealt > 0;
    const launch_shape shape{(uint32_t)(dealt ? l.n_dealt : l.n_blocks), (uint32_t)l.n_tiles, front_blocks(l)};
    int64_t load[256] = {};
    for (uint32_t at = 0; at < shape.n_blocks * shape.n_tiles; ++at) {
        const place p = place_of(shape, launch_group{at % shape.n_blocks, at / shape.n_blocks});
        int64_t chunks = 0;
        for (int w = 0; w < spmm_fmt::WAVES_PER_WG; ++w)
            chunks += (dealt ? l.dealt : l.items)[(p.block * spmm_fmt::WAVES_PER_WG + w) * spmm_fmt::ITEM_WORDS + spmm_fmt::IT_NCHUNKS];
        if (chunks > 0) load[at % 256] += chunks + 8;
    }
    return *std::max_element(load, load + 256) / l.n_tiles;
}

static spmm_plan_t *chunks(const csr &a, int hint)
{
    spmm_options_t o;
    std::memset(&o, 0, sizeof o);
    o.n_hint = hint;
    o.tiles = o.strips = -1;
    spmm_plan_t *p = nullptr;
    REQUIRE(create(a, o, &p) == SPMM_OK);
    return p;
}

// Rows of two lengths: every sixteenth of `many` entries, the others of `few`.
static csr two_lengths(int64_t M, int64_t K, int64_t many, int64_t few)
{
    csr a{M, K};
    for (int64_t i = 0; i < M; ++i) {
        const int64_t n = i % 16 == 0 ? many : few;
        for (int64_t e = 0; e < n; ++e) {
            a.col_idx.push_back((int32_t)(e * K / n));
            a.vals.push_back(1.0f);
        }
        a.row_ptr.push_back((int32_t)a.col_idx.size());
    }
    return a;
}

// One tile at the widths whose bit in `halved` is not set (41 to 64, 97 to 119, 120 to 128 columns), two of half the width at the others.
static void widths(const csr &a, int hint, int halved)
{
    spmm_plan_t *p = chunks(a, hint);
    for (int N : {33, 40, 41, 48, 63, 64, 65, 96, 97, 119, 120, 128, 129}) {
        const spmm_launch_args l = on_columns(p, N)[0];
        const int bit = N > 40 && N <= 64 ? 1 : N > 96 && N < 120 ? 2 : N >= 120 && N <= 128 ? 4 : 0, tile = N > 64 ? 128 : 64;
        std::printf("%lld rows, %d columns: %d of %d\n", (long long)a.M, N, l.n_tiles, l.tile_cols);
        REQUIRE(l.n_tiles == (halved & bit ? 2 : 1) && l.tile_cols == (halved & bit ? tile / 2 : tile));
        REQUIRE(N > 128 || (l.width == N && launched.size() == 1));
    }
    REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
}

int main()
{
    widths(two_lengths(300, 4096, 2000, 40), 64, 7);
    widths(two_lengths(600, 800, 30, 30), 100, 6);     // 75 even blocks: half of the units would be idle
    widths(two_lengths(1024, 2048, 200, 200), 128, 0);  // 256 even blocks
    widths(spread(4096, 0.5, 300, 0.1), 128, 6);
    widths(spread(2048, 0.5, 4096, 0.1), 128, 0);       // more than 512 blocks
    // What a launch of two tiles spares is counted in the order that it gets.  (Block by block, which 97 to 119 and 41 to 64 columns
    // are not, some of these would be spared enough.)
    long taken = 0, left = 0, spared_in_turn = 0;
    for (int64_t M : {230, 300, 340, 400, 440, 480, 520, 600})
        for (int64_t K : {1300, 2500, 4000})
            for (double density : {0.05, 0.1, 0.2}) {
                spmm_plan_t *p = chunks(spread(K, 0.5, M, density), 119);
                spmm_plan_info_t info;
                REQUIRE(spmm_plan_describe(p, &info) == SPMM_OK);
                for (int N : {48, 64, 100, 119, 128}) {
                    const spmm_launch_args l = on_columns(p, N)[0];
                    spmm_launch_args one = on_columns(p, N > 64 ? 96 : 40)[0], two = l;
                    REQUIRE(one.n_tiles == 1 && info.ufk == 8);
                    two.n_dealt = 0;
                    two.n_tiles = 2;
                    two.tile_cols = N > 64 ? 64 : 32;
                    const int64_t before = fullest(one), spared = before - fullest(two);
                    const bool few = info.n_blocks <= 512 && info.k_slices == 1 && info.n_cross == 0;
                    auto enough = [&](int64_t s) { return s >= (N > 64 ? 20 : 120) && s * (info.ufi > 1 && N < 120 ? 4 : 6) >= before; };
                    REQUIRE((l.n_tiles == 2) == (few && enough(spared)));
                    (l.n_tiles == 2 ? taken : left) += 1;
                    two.width = 128;  // block by block
                    two.tile_cols = 64;
                    spared_in_turn += few && l.n_tiles == 1 && enough(before - fullest(two));
                }
                REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
            }
    std::printf("%ld in two tiles, %ld in one, %ld of which two tiles would spare enough block by block\n", taken, left, spared_in_turn);
    REQUIRE(taken > 0 && left > 0 && spared_in_turn > 0);
    std::printf("ok\n");
    return 0;
}
