// Host-side check of the arithmetic with which a workgroup finds its tile
// (hp_tile.hpp), against the plain form of each step:
//   - the bisection of a node's 16 keys against a search from the left, for
//     every tile around every key, with and without padding,
//   - the multiplication that stands for t / parts_per_row, for every number of
//     parts a row can have and tiles around the multiples that a wrong magic number
//     misses first, up to the largest grid,
//   - the 64-bit minimum taken in halves,
//   - which launches are paced.
// usage: walk_lookup <seed>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "hp_tile.hpp"

#define CHECK(c, ...) \
    do { if (!(c)) { std::printf(__VA_ARGS__); std::printf(": %s\n", #c); return 1; } } while (0)

// Rounds of a launch of about `bytes` bytes in tiles of 1 KiB << v, `segs` images of one sample on each destination rank.
static int rounds(int direction, int copies, double bytes, int segs, int64_t row_bytes = 8192, bool sbh = false, int sources = 1,
                  int v = 0, int block = 64) {
    const int64_t per_row = (direction == 0 ? 1 + copies : copies + sources) * row_bytes;
    const int32_t n = (int32_t)(bytes / (double)per_row / segs) + 1;
    std::vector<int32_t> sample(segs, 0), start(segs), len(segs, n);
    for (int i = 0; i < segs; ++i) start[i] = i * (n + 1);
    const hp_layout_t src{sources, 1, 1, 1, 0, 0, 0, 0}, dst{copies, 1, 1, 1, 0, HP_TP_REPLICATE, HP_CP_CONTIGUOUS, sbh ? HP_ROW_SBH : HP_ROW_BSH};
    const hp_token_map_t m{sbh ? 2 : 1, segs * (n + 1), (int32_t)(row_bytes / 2), HP_BF16, segs, sample.data(), start.data(), len.data(), nullptr};
    hp_plan p;
    if (hp::build_host_plan(&src, 1, &dst, &m, 1, &p) != HP_OK || (int)p.segments.size() != segs) return -1;
    return hp::pace_rounds(p, direction, hp::Launch{v, block, 16, 3});
}

static int check_pacing() {
    // where it was measured to gain, fewer rounds the deeper the tree
    for (int c : {2, 3, 4})
        for (int segs : {16, 200, 2000})
            CHECK((rounds(1, c, 600e6, segs) > 0) == (c != 2 || segs > 16), "%d copies, %d segments", c, segs);
    CHECK(rounds(1, 4, 600e6, 9) > rounds(1, 4, 600e6, 99) && rounds(1, 4, 600e6, 99) > rounds(1, 4, 600e6, 999), "levels");
    CHECK(rounds(1, 6, 900e6, 9) > 0 && rounds(1, 6, 900e6, 99) > 0 && rounds(1, 6, 900e6, 999) == 0 && rounds(1, 6, 700e6, 99) == 0, "six copies");
    CHECK(rounds(0, 16, 600e6, 99) > 0 && rounds(0, 16, 600e6, 9) > 0, "forward to sixteen copies");
    // and nowhere else: other counts, small launches, more segments, other shapes and directions, two source copies
    for (int c : {1, 5, 7, 8, 16}) CHECK(rounds(1, c, 2e9, 99) == 0, "%d copies, backward", c);
    for (int c : {1, 2, 3, 4, 8, 13, 15}) CHECK(rounds(0, c, 1e9, 99) == 0, "%d copies, forward", c);
    CHECK(rounds(0, 16, 150e6, 99) == 0 && rounds(0, 16, 1.7e9, 99) == 0, "forward to sixteen copies");
    for (int c : {2, 3, 4}) {
        CHECK(rounds(1, c, 350e6, 99) == 0 && rounds(1, c, 600e6, 5000) == 0, "%d copies", c);
        CHECK(rounds(2, c, 2e9, 99) == 0 && rounds(3, c, 2e9, 99) == 0 && rounds(1, c, 2e9, 99, 8192, false, 2) == 0, "%d copies", c);
        CHECK(rounds(1, c, 2e9, 99, 8192, false, 1, 1) == 0 && rounds(1, c, 2e9, 99, 8192, false, 1, 0, 128) == 0, "%d copies", c);
        // pieces of row-strided rows: whole tiles only
        CHECK(rounds(1, c, 2e9, 99, 8192, true) > 0 && rounds(1, c, 2e9, 99, 1280, true) == 0 && rounds(1, c, 2e9, 99, 3088, true) == 0,
              "%d copies, row-strided", c);
    }
    return 0;
}

int main(int argc, char **argv) {
    std::mt19937_64 rng(argc > 1 ? std::atoll(argv[1]) : 1);
    for (int it = 0; it < 20000; ++it) {
        uint32_t keys[hp::kTreeFanout];
        const int n = 1 + (int)(rng() % hp::kTreeFanout);
        uint32_t k = rng() % 2 ? 0 : (uint32_t)(rng() % 0x70000000u);
        for (int j = 0; j < hp::kTreeFanout; ++j) {
            keys[j] = j < n ? k : UINT32_MAX;
            k += 1 + (uint32_t)(rng() % (rng() % 4 ? 5u : 0x800000u));
        }
        for (int j = 0; j < n; ++j)
            for (int64_t d = -1; d <= 1; ++d) {
                const int64_t tile = (int64_t)keys[j] + d;
                if (tile < keys[0] || tile > 0x7fffffff) continue;
                uint32_t index, key, want = 0;
                hp::search_node(keys, (uint32_t)tile, index, key);
                while (want + 1 < hp::kTreeFanout && keys[want + 1] <= (uint32_t)tile) ++want;
                CHECK(index == want && key == keys[want], "node %d key %d tile %lld", it, j, (long long)tile);
            }
    }
    const uint32_t most = (1u << 24) / hp::tile_bytes_of(0) + 1;           // rows of up to 16 MiB, and one more
    for (uint32_t d = 1; d <= most; ++d) {
        hp::KParams p{};
        p.parts_per_row = d;
        hp::set_parts(p);
        auto row = [&](uint32_t t) { return (uint32_t)((uint64_t)t * p.part_magic >> 31 >> p.part_shift); };
        const uint32_t last = 0x7fffffffu, top = last / d * d;
        const uint32_t some = (uint32_t)(rng() % (last / d + 1)) * d;
        for (uint32_t m : {0u, d, some, top})
            for (int64_t t = (int64_t)m - 1; t <= (int64_t)m + 1; ++t)
                if (t >= 0 && t <= last) CHECK(row((uint32_t)t) == (uint32_t)t / d, "parts %u tile %lld", d, (long long)t);
        CHECK(row(last) == last / d, "parts %u, last tile", d);
    }
    for (uint64_t left : {(uint64_t)0, (uint64_t)1, (uint64_t)1023, (uint64_t)1024, (uint64_t)1025, (uint64_t)UINT32_MAX,
                          (uint64_t)1 << 32, ((uint64_t)1 << 32) + 1, ((uint64_t)5 << 32) + 1024})
        CHECK(hp::clip(left, 1024) == (left < 1024 ? left : 1024), "left %llu", (unsigned long long)left);
    if (check_pacing()) return 1;
    std::printf("ok\n");
    return 0;
}
