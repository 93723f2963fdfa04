// Host-side walk of launches that cut row-strided segments by bytes, with the code
// the GPU runs (hp_tile.hpp): built by tests/test_cut_rows.py with UBSan.  For random
// plans, every tile size that has such launches and both chunk sizes it checks
// that the tiles partition the segments in order, that each is whole but the
// last of its segment, and that every byte has the destination offset that its row and
// column give, which is where the same plan's row by row launch puts it.
// usage: walk_cut <seed> <plans>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "hp_tile.hpp"

static int it, v;
static uint32_t tile;
#define CHECK(c) do { if (!(c)) { std::printf("plan %d variant %d tile %u: %s\n", it, v, tile, #c); return 1; } } while (0)

template <uint32_t UNIT>
static int walk(const hp_plan &p, const uint32_t *tree, long *tiles) {
    hp::KParams k = hp::kernel_params(p, v, p.dsegs.data(), tree, true);
    hp::set_row_chunks(k, UNIT);
    CHECK(hp::seg_kinds(k, (uint64_t)p.dst_stride) == hp::kCutRows);
    size_t seg = 0;
    uint64_t covered = 0;
    for (tile = 0; tile < p.cut_tiles[v]; ++tile, ++*tiles) {
        const hp::TileView t = hp::locate_tile(k, tile);
        while (covered == (uint64_t)p.dsegs[seg].n_rows * k.row_bytes) { ++seg; covered = 0; CHECK(seg < p.dsegs.size()); }
        const hp::Seg &s = p.dsegs[seg];
        CHECK(t.src_buf == s.src_buf && t.dst_buf0 == s.dst_buf0 && t.src_copies == s.src_copies && t.pitch_rows == s.pitch_rows);
        CHECK(t.src_off == s.src_off + covered && t.nbytes % UNIT == 0);
        CHECK(t.nbytes == std::min<uint64_t>(k.tile_bytes, (uint64_t)s.n_rows * k.row_bytes - covered));
        for (uint32_t i = 0; i < t.nbytes / UNIT; ++i) {
            const hp::ChunkView c = hp::cut_chunk<UNIT>(k, t, i);
            const uint64_t off = covered + (uint64_t)i * UNIT, row = off / k.row_bytes;
            CHECK(c.src == i * UNIT && c.over == 0);
            CHECK(t.dst_off + c.dst == s.dst_off + row * s.pitch_rows * k.row_bytes + off % k.row_bytes);
            CHECK(t.dst_off + c.dst + UNIT <= (uint64_t)p.dst_rows_per_buf * k.row_bytes);
        }
        covered += t.nbytes;
    }
    CHECK(seg + 1 == p.dsegs.size() && covered == (uint64_t)p.dsegs[seg].n_rows * k.row_bytes);
    return 0;
}

// Rows that are not whole lines: chunks that are there cover every byte of every row, and none of another; they lie on
// 16-byte pieces of the destination but where they were moved to an end of their row.
// What counts of each, between over and end, is every byte once.
template <uint32_t UNIT>
static int walk_padded(const hp_plan &p, const uint32_t *tree, uint64_t dst_base, long *tiles) {
    hp::KParams k = hp::kernel_params(p, v, p.dsegs.data(), tree, true);
    hp::set_row_chunks(k, UNIT);
    CHECK(hp::seg_kinds(k, (uint64_t)p.dst_stride) == hp::kPaddedRows);
    std::vector<std::vector<uint8_t>> seen(p.dsegs.size());
    for (size_t i = 0; i < seen.size(); ++i) seen[i].assign((size_t)p.dsegs[i].n_rows * k.row_bytes, 0);
    const uint64_t lines = (uint64_t)hp::cut_row_lines(p.row_bytes);
    size_t seg = 0;
    uint64_t done = 0;                                          // lines of the segment
    for (tile = 0; tile < p.cut_tiles[v]; ++tile, ++*tiles) {
        const hp::TileView t = hp::locate_tile(k, tile);
        while (done == p.dsegs[seg].n_rows * lines) { ++seg; done = 0; CHECK(seg < p.dsegs.size()); }
        const hp::Seg &s = p.dsegs[seg];
        const uint64_t row0 = done / lines;
        CHECK(t.src_off == s.src_off + row0 * k.row_bytes && t.dst_off == s.dst_off + row0 * s.pitch_rows * k.row_bytes);
        CHECK(t.src_buf == s.src_buf && t.dst_buf0 == s.dst_buf0 && t.col == (done - row0 * lines) * 128);
        CHECK(t.nbytes == std::min<uint64_t>(k.tile_bytes, (s.n_rows * lines - done) * 128));
        for (uint32_t i = 0; i < t.nbytes / UNIT; ++i) {
            hp::ChunkView c;
            const bool there = hp::padded_chunk<UNIT>(k, t, (uint32_t)(dst_base + t.dst_off), i, c);
            const uint64_t at = row0 * k.row_bytes + c.src, row = at / k.row_bytes, in_row = at % k.row_bytes;
            CHECK(row < s.n_rows && in_row + UNIT <= k.row_bytes);      // whether there or not: it is read
            CHECK(t.dst_off + c.dst == s.dst_off + row * s.pitch_rows * k.row_bytes + in_row);
            if (!there) continue;
            CHECK((dst_base + t.dst_off + c.dst) % UNIT == 0 || in_row == 0 || in_row + UNIT == k.row_bytes);
            CHECK(c.over < c.end && c.end <= UNIT && c.over % p.elem_bytes == 0 && c.end % p.elem_bytes == 0);
            for (uint32_t b = c.over; b < c.end; ++b) CHECK(!seen[seg][at + b]++);
        }
        done += t.nbytes / 128;
    }
    CHECK(seg + 1 == p.dsegs.size() && done == p.dsegs[seg].n_rows * lines);
    for (const auto &x : seen)
        for (uint8_t y : x) CHECK(y);
    return 0;
}

int main(int argc, char **argv) {
    std::mt19937_64 rng(argc > 1 ? std::atoll(argv[1]) : 1);
    const int plans = argc > 2 ? std::atoi(argv[2]) : 60;
    auto R = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
    int done = 0;
    long tiles = 0;
    for (it = 0; done < plans && it < 100 * plans; ++it) {
        const hp_layout_t src{R(1, 2), 1, R(1, 3), 1, 0, 0, 0, 0};
        const hp_layout_t dst{R(1, 9), R(1, 2), 1, 1, 0, R(0, 1), R(0, 1), HP_ROW_SBH};
        const int hiddens[] = {64, 192, 320, 448, 640, 1088, 1280, 2304, 65344}, ragged[] = {1025, 130, 695, 1544, 2305, 65535};
        const int batch = R(2, 5), seq = 2 * dst.cp * dst.tp * R(1, 12), f32 = R(0, 1);
        std::vector<int32_t> smp, st, ln;
        for (int b = 0; b < batch; ++b)
            for (int pos = R(0, 6); pos < seq;) {
                const int len = std::min(seq - pos, R(1, 1 + seq / 3));
                smp.push_back(b); st.push_back(pos); ln.push_back(len);
                pos += len + R(0, 4);
            }
        const bool padded = R(0, 1);
        const int hidden = padded ? (R(0, 19) ? ragged[R(0, 4)] : ragged[5] >> f32) : R(0, 19) ? hiddens[R(0, 7)] : hiddens[8] >> f32;
        const hp_token_map_t m{batch, seq, hidden, f32, (int32_t)smp.size(), smp.data(), st.data(), ln.data(), nullptr};
        hp_plan p;
        if (hp::build_host_plan(&src, 1, &dst, &m, 1, &p) != HP_OK || p.segments.empty()) continue;
        ++done;
        uint32_t *tree = (uint32_t *)std::aligned_alloc(64, (p.tree.size() * 4 + 63) / 64 * 64 + 64);
        std::copy(p.tree.begin(), p.tree.end(), tree);
        for (v = 0; v < hp::kTileVariants; ++v) {
            tile = 0;
            const int64_t bytes = hp::tile_bytes_of(v);
            if (padded) {
                CHECK((p.cut_tiles[v] > 0) == (v < hp::kCutVariants));
                const uint64_t e = (uint64_t)p.elem_bytes, bases[] = {0, e, 64, 126 / e * e};
                if (p.cut_tiles[v])
                    if (walk_padded<16>(p, tree, bases[it % 4], &tiles) || (!f32 && walk_padded<8>(p, tree, bases[it % 4], &tiles))) return 1;
                continue;
            }
            CHECK((p.cut_tiles[v] > 0) == (v < hp::kCutVariants && p.row_bytes % bytes != 0 && bytes % p.row_bytes != 0));
            CHECK(p.cut_tiles[v] <= p.n_tiles(v));
            if (!p.cut_tiles[v]) continue;
            if (walk<16>(p, tree, &tiles) || (!f32 && walk<8>(p, tree, &tiles))) return 1;
        }
        std::free(tree);
    }
    std::printf("plans %d\n", done);
    return done == plans && tiles > 1000 ? 0 : 2;
}
