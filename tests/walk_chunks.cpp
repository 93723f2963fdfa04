// Host-side walk of every lane chunk of every tile, with the code the GPU runs
// (hp_tile.hpp): built by tests/test_chunks_host.py with ASan + UBSan.  For random
// plans, every tile size, several alignments of the destination buffer and the
// lane chunks of each direction (16 bytes; 8 bytes of bf16 gradients) it checks that
//   - the tiles with their ends moved to lines still partition the segments,
//   - inside a run they begin on a line of the destination,
//   - the chunks of a tile, less the bytes a moved chunk shares with the one
//     before it, cover every byte of it once, and none leaves its run,
//   - every byte has the destination offset that its row and column give.
// usage: walk_chunks <seed> <plans>
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "hp_tile.hpp"

static int it, v;
static uint32_t tile;
#define CHECK(c)                                                                                    \
    do {                                                                                            \
        if (!(c)) { std::printf("plan %d variant %d tile %u: %s\n", it, v, tile, #c); return false; } \
    } while (0)

// Checks one tile's walk; `seg_off` = source bytes of the segment before the tile.
template <uint32_t UNIT, uint32_t ELEM, bool DENSE>
static bool walk_tile(const hp::KParams &k, const hp::TileView &t, const hp::Seg &s, uint64_t seg_off) {
    std::vector<uint8_t> seen(t.nbytes, 0);
    uint32_t n, whole;
    hp::count_chunks<UNIT, DENSE>(k, t, n, whole);
    auto at = [&](uint64_t in_tile) {                       // destination offset of a byte, from the definition
        const uint64_t off = seg_off + in_tile, row = off / k.row_bytes;
        return s.dst_off + row * s.pitch_rows * k.row_bytes + off % k.row_bytes;
    };
    auto cover = [&](const hp::ChunkView &c, uint32_t len) {
        CHECK(c.src + len <= t.nbytes && c.over < len);
        for (uint32_t b = 0; b < len; ++b) CHECK(t.dst_off + c.dst + b == at(c.src + b));
        for (uint32_t b = c.over; b < len; ++b) CHECK(!seen[c.src + b]++);
        for (uint32_t b = 0; b < c.over; ++b) CHECK(seen[c.src + b] == 1);
        return true;
    };
    if (n == 0) {
        CHECK((DENSE ? t.nbytes : k.row_bytes) < UNIT);
        for (uint32_t i = 0; i < t.nbytes / ELEM; ++i)
            if (!cover(hp::element_at<ELEM>(k, t, i), ELEM)) return false;
    }
    CHECK(whole <= n && n - whole <= 1);
    for (uint32_t i = 0; i < n; ++i) {
        const hp::ChunkView c = hp::chunk_at<UNIT, DENSE, true>(k, t, i);
        CHECK(c.over % ELEM == 0);
        if (i < whole) {
            const hp::ChunkView d = hp::chunk_at<UNIT, DENSE, false>(k, t, i);
            CHECK(d.src == c.src && d.dst == c.dst && d.over == c.over && (!DENSE || c.over == 0));
        }
        if (!cover(c, UNIT)) return false;
    }
    for (uint8_t x : seen) CHECK(x == 1);
    return true;
}

template <uint32_t UNIT, uint32_t ELEM>
static bool walk_plan(const hp_plan &p, const uint32_t *tree, uint64_t dst_base) {
    hp::KParams k = hp::kernel_params(p, v, p.dsegs.data(), tree);
    hp::set_row_chunks(k, UNIT);
    size_t seg = 0;
    uint64_t covered = 0;
    for (tile = 0; tile < p.n_tiles(v); ++tile) {
        hp::TileView t = hp::locate_tile(k, tile);
        hp::align_tile(t, dst_base);
        if (t.nbytes == 0) continue;                        // its run ended within the tile before it
        while (covered == (uint64_t)p.dsegs[seg].n_rows * k.row_bytes) { ++seg; covered = 0; CHECK(seg < p.dsegs.size()); }
        const hp::Seg &s = p.dsegs[seg];
        CHECK(t.src_off == s.src_off + covered && t.nbytes <= std::max(k.tile_bytes, k.row_bytes) + hp::kLineBytes);
        const bool run_start = s.pitch_rows == 1 ? covered == 0 : covered % k.row_bytes == 0;
        if (t.pitch_rows == 1 && !run_start) CHECK((dst_base + t.dst_off) % hp::kLineBytes == 0);
        const bool ok = t.pitch_rows == 1 ? walk_tile<UNIT, ELEM, true>(k, t, s, covered)
                                          : walk_tile<UNIT, ELEM, false>(k, t, s, covered);
        if (!ok) return false;
        covered += t.nbytes;
    }
    while (seg < p.dsegs.size() && covered == (uint64_t)p.dsegs[seg].n_rows * k.row_bytes) { ++seg; covered = 0; }
    CHECK(seg == p.dsegs.size() && covered == 0);
    return true;
}

// The runs of hp_text_grads: a partition of every buffer's rows in which exactly
// the segments' rows are image rows; whole: one dense run for each first copy.
static bool check_runs(const hp_plan &p) {
    v = -1; tile = 0;
    for (int whole = 0; whole < 2; ++whole) {
        std::vector<std::vector<int>> rows((size_t)p.n_dst_bufs, std::vector<int>((size_t)p.dst_rows_per_buf, -1));
        const std::vector<hp::Seg> runs = hp::dst_runs(p, whole != 0);
        if (whole) CHECK(runs.size() == (size_t)(p.n_dst_bufs / p.dst_copies));
        for (const hp::Seg &r : runs) {
            CHECK(r.n_rows > 0 && r.src_off == r.dst_off && r.src_buf == r.dst_buf0);
            CHECK(r.pitch_rows == (whole ? 1 : p.dst_stride));
            for (uint32_t i = 0; i < r.n_rows; ++i) {
                int &cell = rows[r.dst_buf0][r.dst_off / (uint64_t)p.row_bytes + (uint64_t)i * r.pitch_rows];
                CHECK(cell == -1);
                cell = (int)r.src_copies;
            }
        }
        for (const hp_segment_t &s : p.segments)
            for (int64_t i = 0; i < s.n_rows; ++i) {
                int &cell = rows[s.dst_buf0][s.dst_row0 + i * s.dst_row_stride];
                CHECK(cell == (whole ? 0 : 1));
                cell = 0;
            }
        for (int b = 0; b < p.n_dst_bufs; ++b)
            for (int x : rows[b]) CHECK(x == (b % p.dst_copies ? -1 : 0));
    }
    return true;
}

int main(int argc, char **argv) {
    std::setvbuf(stdout, nullptr, _IONBF, 0);
    std::mt19937_64 rng(argc > 1 ? std::atoll(argv[1]) : 1);
    const int plans = argc > 2 ? std::atoi(argv[2]) : 60;
    auto R = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
    int done = 0;
    for (it = 0; done < plans && it < 100 * plans; ++it) {
        hp_layout_t src{1, 1, R(1, 4), 1, 0, 0, 0, 0};
        hp_layout_t dst{R(1, 3), R(1, 2), 1, 1, 0, R(0, 1), R(0, 1), R(0, 1)};
        const int batch = R(1, 3), seq = 2 * dst.cp * dst.tp * R(1, 10);
        const int hiddens[] = {1, 2, 3, 5, 7, 8, 9, 15, 33, 64, 100, 513, 1001};
        std::vector<int32_t> smp, st, ln;
        for (int b = 0; b < batch; ++b)
            for (int pos = R(0, 6); pos < seq;) {
                const int len = std::min(seq - pos, R(1, 1 + seq / 3));
                smp.push_back(b); st.push_back(pos); ln.push_back(len);
                pos += len + R(0, 4);
            }
        const int f32 = R(0, 1);
        hp_token_map_t m{batch, seq, hiddens[R(0, 12)], f32, (int32_t)smp.size(), smp.data(), st.data(), ln.data(), nullptr};
        hp_plan p;
        if (hp::build_host_plan(&src, 1, &dst, &m, 1, &p) != HP_OK || p.segments.empty()) continue;
        ++done;
        if (!check_runs(p)) return 1;
        uint32_t *tree = (uint32_t *)std::aligned_alloc(64, (p.tree.size() * 4 + 63) / 64 * 64 + 64);
        std::copy(p.tree.begin(), p.tree.end(), tree);
        const uint64_t e = (uint64_t)p.elem_bytes, bases[] = {0, e, 16, 126 / e * e};
        for (v = 0; v < hp::kTileVariants; v += 1 + v % 2)
            for (uint64_t base : bases) {
                if (!(f32 ? walk_plan<16, 4>(p, tree, base) : walk_plan<16, 2>(p, tree, base))) return 1;
                if (!f32 && !walk_plan<8, 2>(p, tree, base)) return 1;
            }
        std::free(tree);
    }
    std::printf("plans %d\n", done);
    return done == plans ? 0 : 2;
}
