// Host-side checks of the rules by which launches of row-strided plans are cut and
// shaped: built by tests/test_cut_rules.py with UBSan.
// usage: walk_rules <check> <seed> <plans>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <random>
#include <vector>

#include "hp_tile.hpp"

static int it;
static long allocations;
void *operator new(size_t n) {
    ++allocations;
    if (void *p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
#define CHECK(c) do { if (!(c)) { std::printf("plan %d: %s\n", it, #c); return 1; } } while (0)

// A plan of `samples` samples a position, `rows` rows in `images` images in each.
static int make(hp_plan &p, int tp_src, int tp, int samples, int hidden, int f32, int64_t rows, int images, int order = HP_ROW_SBH) {
    const hp_layout_t src{tp_src, 1, 1, 1, 0, 0, 0, 0}, dst{tp, 1, 1, 1, 0, 0, 0, order};
    std::vector<int32_t> smp, st, ln;
    int64_t seq = 1;
    for (int b = 0; b < samples; ++b) {
        int64_t at = 0;
        for (int k = 0; k < images; ++k) {
            const int64_t n = (k + 1) * rows / images - k * rows / images;
            smp.push_back(b); st.push_back((int32_t)at); ln.push_back((int32_t)n);
            at += n + 1;
        }
        seq = at;
    }
    const hp_token_map_t m{samples, (int32_t)seq, hidden, f32, (int32_t)smp.size(), smp.data(), st.data(), ln.data(), nullptr};
    return hp::build_host_plan(&src, 1, &dst, &m, 1, &p);
}

// What a launch asks is answered from what the plan was made with: no rule reads the segments again, which would
// cost every launch of a plan of many images a walk.
static int once(std::mt19937_64 &rng, int plans) {
    auto R = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
    long cut = 0;
    for (it = 0; it < plans; ++it) {
        const int hiddens[] = {192, 1025, 1088, 1280, 2305, 1544, 2304, 695};
        hp_plan p;
        CHECK(make(p, R(1, 2), R(1, 9), R(2, 4), hiddens[R(0, 7)], R(0, 1), 400 << R(0, 7), R(1, 40)) == HP_OK);
        bool was[3][hp::kTileVariants];
        int pace[3];
        const hp::Launch one{0, 64, 16, 3};
        for (int d = 0; d < 3; ++d) {
            pace[d] = hp::pace_rounds(p, d, one);
            for (int v = 0; v < hp::kTileVariants; ++v) cut += was[d][v] = hp::cuts_launch(p, d, v);
        }
        for (hp_segment_t &s : p.segments) s.n_rows = INT32_MAX;
        for (int d = 0; d < 3; ++d) {
            CHECK(pace[d] == hp::pace_rounds(p, d, one));
            for (int v = 0; v < hp::kTileVariants; ++v) CHECK(was[d][v] == hp::cuts_launch(p, d, v));
        }
    }
    CHECK(cut > plans);
    return 0;
}

// Plans are made at step rate: what a plan needs for rows that can be cut is made in place, with no allocation but
// the keys it is made from.  (At 1000 segments the trees of the four tile sizes, put together in lists of their own,
// were a fifth of the time of a plan.)
static int made_in_place(std::mt19937_64 &rng, int plans) {
    for (it = 0; it < plans; ++it) {
        const int images = 1 + (int)(rng() % 300);
        long n[2];
        for (int cut = 0; cut < 2; ++cut) {
            hp_plan p;
            const long before = allocations;
            CHECK(make(p, 1, 4, 4, cut ? 2304 : 4096, 0, 16 * images, images) == HP_OK);
            n[cut] = allocations - before;
            CHECK((p.cut_tiles[0] > 0) == (cut == 1));
        }
        CHECK(n[1] <= n[0] + 1);
    }
    return 0;
}

// A plan whose forward moves about `mb` megabytes, in [S,B,H] order with four samples a position.
static int sized(hp_plan &p, int tp, int row, double mb, int f32 = 0) {
    return make(p, 1, tp, 4, row / (f32 ? 4 : 2), f32, (int64_t)(mb * 1e6 / (1 + tp) / row / 4), 8);
}

// Shapes that suit whole tiles are for launches that have them: rows that leave tiles partly empty and are not cut there
// keep the shape that they had.
static int shapes() {
    struct Case { int tp, row; double mb; bool small; };
    for (const Case &c : {Case{4, 10240, 160, true}, Case{4, 10240, 190, true}, Case{4, 10240, 210, true}, Case{4, 3712, 300, false}, Case{4, 3584, 220, false}, Case{4, 3712, 700, true}, Case{4, 3968, 300, true},
                          Case{12, 3584, 300, false}, Case{16, 3712, 200, false}, Case{16, 3712, 700, true}, Case{14, 4608, 300, true},
                          Case{8, 3712, 120, false}, Case{8, 3712, 300, true}, Case{8, 2560, 120, true}, Case{4, 8192, 300, true}}) {
        hp_plan p;
        ++it;
        CHECK(sized(p, c.tp, c.row, c.mb) == HP_OK);
        CHECK((p.fwd.tile_variant == 0) == c.small);
    }
    for (const Case &c : {Case{1, 3712, 60, false}, Case{1, 7552, 60, false}, Case{3, 3968, 60, false}, Case{8, 3712, 100, false},
                          Case{1, 2304, 60, true}, Case{1, 4608, 60, true}, Case{8, 2304, 100, true}}) {      // accumulating, in 4 KiB
        hp_plan p;
        ++it;
        CHECK(sized(p, c.tp, c.row, c.mb) == HP_OK);
        CHECK((p.acc.tile_variant == 2 && p.acc.waves_per_cu > 0) == c.small);
    }
    return 0;
}

// Launches that were slower when they were cut: groups of rows forward in 1 KiB tiles, groups that leave much less of a
// tile empty, one row in an 8 KiB tile to two copies.
static int cuts() {
    struct Case { int tp, row; double mb; int direction, variant; bool cut; };
    for (const Case &c : {Case{4, 600, 120, 0, 0, false}, Case{3, 700, 170, 0, 0, false}, Case{4, 600, 300, 0, 1, true}, Case{4, 600, 120, 1, 0, true},
                          Case{8, 500, 120, 0, 1, false}, Case{2, 600, 120, 0, 3, true}, Case{2, 4608, 150, 0, 3, false}, Case{2, 4608, 60, 0, 3, true},
                          Case{2, 9216, 150, 0, 3, true}, Case{2, 2304, 150, 0, 3, true}, Case{3, 4608, 150, 0, 3, true}, Case{4, 2050, 120, 0, 0, true}}) {
        hp_plan p;
        ++it;
        CHECK(sized(p, c.tp, c.row, c.mb) == HP_OK);
        CHECK(hp::cuts_launch(p, c.direction, c.variant) == c.cut);
    }
    return 0;
}

// A grid of 2^32 work-items is refused.  Where tiles of lines are more of them than the row by row launch has, which the
// starting shapes were checked with, the largest launches go row by row: backward from two copies in rows of 900 bytes,
// 9 lines of 8 a tile against one row a tile.
static int grids() {
    long near = 0;
    for (int64_t rows : {1000, 900000, 1000000, 15000000, 15700000, 16700000}) {
        hp_plan p;
        ++it;
        CHECK(make(p, 2, 2, 4, 450, 0, rows, 1) == HP_OK);
        CHECK(p.bwd.tile_variant == 0 && p.bwd.block == 64);
        const uint64_t cut = (uint64_t)p.cut_tiles[0] * 64, plain = (uint64_t)p.n_tiles(0) * 64;
        near += cut >= 1ull << 32 && plain < 1ull << 32;
        CHECK((hp::cuts_launch(p, 1, 0) ? cut : plain) < 1ull << 32);
        CHECK(hp::cuts_launch(p, 1, 0) == (rows < 1000000));
    }
    CHECK(near == 3);
    return 0;
}

// hp_text_grads of samples whose images lie alike takes their bands, which are as many as one sample has runs, where a copy
// of everything was taken for as many as all samples have; scattered images change nothing.
static int alike(std::mt19937_64 &rng) {
    for (it = 0; it < 8; ++it) {
        const bool scattered = it & 1, last_differs = it & 2;
        const int samples = 4, images = 60, copies = 2, dp = it & 4 ? 2 : 1;
        const hp_layout_t src{1, 1, 1, 1, 0, 0, 0, 0}, dst{copies, 1, dp, 1, 0, 0, 0, HP_ROW_SBH};
        std::vector<int32_t> smp, st, ln;
        for (int b = 0; b < samples * dp; ++b)
            for (int k = 0; k < images; ++k) {
                smp.push_back(b);
                st.push_back(20 * k + (scattered ? (int)(rng() % 8) : 0));
                ln.push_back(10 + (last_differs && k == images - 1 && b == samples * dp - 1));
            }
        // saves some 40 MB of traffic: worth three launches
        const hp_token_map_t m{samples * dp, 20 * images + 20, 2048, 0, (int32_t)smp.size(), smp.data(), st.data(), ln.data(), nullptr};
        hp_plan p;
        CHECK(hp::build_host_plan(&src, 1, &dst, &m, 1, &p) == HP_OK);
        bool whole;
        const std::vector<hp::Seg> runs = hp::text_runs(p, &whole);
        if (scattered) CHECK(whole && runs.size() == (size_t)dp);
        else if (!last_differs) CHECK(!whole && runs.size() == (size_t)(2 * images) * dp);
        else CHECK(whole);                                   // one that differs: as before
    }
    return 0;
}

int main(int argc, char **argv) {
    if (argc < 4) return 2;
    std::mt19937_64 rng(std::atoll(argv[2]));
    const int plans = std::atoi(argv[3]);
    int rc = 2;
    if (!std::strcmp(argv[1], "once")) rc = once(rng, plans);
    if (!std::strcmp(argv[1], "made_in_place")) rc = made_in_place(rng, plans);
    if (!std::strcmp(argv[1], "shapes")) rc = shapes();
    if (!std::strcmp(argv[1], "cuts")) rc = cuts();
    if (!std::strcmp(argv[1], "grids")) rc = grids();
    if (!std::strcmp(argv[1], "alike")) rc = alike(rng);
    if (rc == 0) std::printf("plans %d\n", plans);
    return rc;
}
