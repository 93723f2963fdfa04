// Host-side check of the arithmetic with which a workgroup finds its tile
// (hp_tile.hpp), against the plain form of each step:
//   - the bisection of a node's 16 keys against a search from the left, for
//     every tile around every key, with and without padding,
//   - the multiplication that stands for t / parts_per_row, for every number of
//     parts a row can have and tiles around the multiples that a wrong magic number
//     misses first, up to the largest grid,
//   - the 64-bit minimum taken in halves.
// usage: walk_lookup <seed>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "hp_tile.hpp"

#define CHECK(c, ...) \
    do { if (!(c)) { std::printf(__VA_ARGS__); std::printf(": %s\n", #c); return 1; } } while (0)

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
    std::printf("ok\n");
    return 0;
}
