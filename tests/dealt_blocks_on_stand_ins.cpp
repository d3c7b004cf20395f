// The order in which a chunk plan's blocks are dealt to the compute units (deal_blocks in spmm_api.cpp), as spmm_execute hands
// it to the launcher, on the stand-ins of host_sources_on_stand_ins.cpp.
#define main main_of_host_sources
#include "host_sources_on_stand_ins.cpp"
#undef main

#include <map>

constexpr size_t WORDS = (size_t)spmm_fmt::WAVES_PER_WG * spmm_fmt::ITEM_WORDS;

static int64_t weight(const uint32_t *block)
{
    int64_t chunks = 0;
    for (int w = 0; w < spmm_fmt::WAVES_PER_WG; ++w) chunks += block[w * spmm_fmt::ITEM_WORDS + spmm_fmt::IT_NCHUNKS];
    return chunks;
}

// Whether the launch on N columns of a chunk plan of `a`, made for `hint`, has dealt blocks: then every block once, idle ones
// between, and the fullest of the 256 units with less to do than in the plan's own order.
static bool dealt(const csr &a, int hint, int N)
{
    static float word;
    spmm_options_t o;
    std::memset(&o, 0, sizeof o);
    o.n_hint = hint;
    o.tiles = o.strips = -1;
    spmm_plan_t *p = nullptr;
    REQUIRE(create(a, o, &p) == SPMM_OK);
    launched.clear();
    REQUIRE(spmm_execute(p, &word, N, &word, nullptr) == SPMM_OK && !launched.empty());
    const spmm_launch_args args = launched[0];
    if (args.n_dealt > 0) {
        REQUIRE(args.n_tiles == 1 && args.n_blocks > 256 && args.n_dealt >= args.n_blocks);
        std::map<std::vector<uint32_t>, int> own;
        int64_t before[256] = {}, now[256] = {};
        for (int32_t b = 0; b < args.n_blocks; ++b) {
            const uint32_t *at = args.items + (size_t)b * WORDS;
            ++own[std::vector<uint32_t>(at, at + WORDS)];
            before[b % 256] += weight(at);
        }
        for (int32_t b = 0; b < args.n_dealt; ++b) {
            const uint32_t *at = args.dealt + (size_t)b * WORDS;
            now[b % 256] += weight(at);
            bool idle = true;
            for (int w = 0; w < spmm_fmt::WAVES_PER_WG; ++w) {
                const uint32_t *it = at + w * spmm_fmt::ITEM_WORDS;
                idle = idle && it[spmm_fmt::IT_NWINS] == 0 && it[spmm_fmt::IT_FLAGS] == spmm_fmt::FLAG_IDLE;
            }
            if (idle) continue;
            const auto found = own.find(std::vector<uint32_t>(at, at + WORDS));
            REQUIRE(found != own.end() && --found->second >= 0);
        }
        for (const auto &left : own) REQUIRE(left.second == 0);
        REQUIRE(*std::max_element(now, now + 256) < *std::max_element(before, before + 256));
    }
    REQUIRE(spmm_plan_destroy(p) == SPMM_OK);
    return args.n_dealt > 0;
}

int main()
{
    const csr uneven = spread(4096, 0.5), few = spread(512, 0.5);
    REQUIRE(dealt(uneven, 64, 64) && dealt(uneven, 64, 40) && dealt(uneven, 64, 128));
    REQUIRE(dealt(spread(2048, 0.5), 64, 64));                  // a few more than 256 blocks
    REQUIRE(dealt(spread(4096, 0.5, 2048, 0.1), 32, 32));       // chunks of 16 columns
    REQUIRE(dealt(spread(5000, 0.5, 700, 0.1), 100, 100));      // panels of two rows
    REQUIRE(!dealt(uneven, 64, 256));                           // two column tiles
    REQUIRE(!dealt(matrix(1024, 4096, 10, 0), 64, 64));          // rows of one length
    REQUIRE(!dealt(few, 64, 64));                               // a block per unit at most
    REQUIRE(!dealt(spread(4096, 0.5, 16384, 0.02), 64, 64));    // more than the chip holds
    std::printf("ok\n");
    return 0;
}
