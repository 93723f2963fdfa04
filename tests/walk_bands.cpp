// Host-side walk of the bands that hp_text_grads takes in [S,B,H] order, with the
// code the GPU runs (hp_tile.hpp): built by tests/test_text_bands.py with UBSan.  For
// random plans and every tile size the tiles of the bands cover every byte of
// every first copy once, and their samples are image exactly where a segment is.
// usage: walk_bands <seed> <plans>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "hp_tile.hpp"

static int it, v;
#define CHECK(c) do { if (!(c)) { std::printf("plan %d variant %d: %s\n", it, v, #c); return 1; } } while (0)

// One launch of all bands in tiles of 1 KiB << v (a tree of one node a level at most here: the bands are looked up one by one).
template <hp::SegKinds KINDS>
static int walk(const hp_plan &p, const std::vector<hp::Seg> &bands, hp::KParams k, const std::vector<std::vector<int>> &image) {
    std::vector<std::vector<int>> seen((size_t)p.n_dst_bufs, std::vector<int>((size_t)p.dst_rows_per_buf * p.row_bytes, 0));
    for (const hp::Seg &b : bands) {
        CHECK(b.pitch_rows == 1 && b.n_rows % k.band_samples == 0 && b.dst_off % (k.band_samples * p.row_bytes) == 0);
        const uint64_t n = hp::tiles_of(b.n_rows, k.band_samples, p.row_bytes, k.tile_bytes);
        k.n_levels = 1;
        for (uint32_t &key : k.root) key = UINT32_MAX;
        k.root[0] = 0;
        for (uint64_t tile = 0; tile < n; ++tile) {
            const hp::TileView t = hp::locate_tile<KINDS, true>(k, &b, nullptr, (uint32_t)tile);
            for (uint32_t i = 0; i < t.nbytes; ++i) {
                const uint64_t at = t.dst_off + i, row = at / p.row_bytes;
                const uint32_t in_tile = KINDS == hp::kRowGroups ? i / k.row_bytes : 0u;
                CHECK(at < seen[b.dst_buf0].size() && !seen[b.dst_buf0][at]++);
                CHECK((t.row + in_tile) == row - b.dst_off / p.row_bytes);
                const uint32_t sample = hp::band_sample(k, hp::band_sample(k, t.row) + in_tile);
                CHECK((int)(b.src_copies >> sample & 1u) == image[b.dst_buf0][row]);
            }
        }
    }
    for (int j = 0; j < p.n_dst_bufs; j += p.dst_copies)
        for (int x : seen[j]) CHECK(x == 1);
    return 0;
}

int main(int argc, char **argv) {
    std::mt19937_64 rng(argc > 1 ? std::atoll(argv[1]) : 1);
    const int plans = argc > 2 ? std::atoi(argv[2]) : 60;
    auto R = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
    int done = 0;
    for (it = 0; done < plans && it < 100 * plans; ++it) {
        const hp_layout_t src{1, 1, R(1, 3), 1, 0, 0, 0, 0};
        const hp_layout_t dst{R(1, 3), R(1, 2), 1, 1, 0, R(0, 1), R(0, 1), HP_ROW_SBH};
        const int batches[] = {2, 3, 4, 5, 31, 32}, hiddens[] = {1, 3, 8, 100, 511, 513, 1200};
        const int batch = batches[R(0, 5)], seq = 2 * dst.cp * dst.tp * R(1, 10);
        std::vector<int32_t> smp, st, ln;
        for (int b = 0; b < batch; ++b)
            for (int pos = R(0, 6); pos < seq;) {
                const int len = std::min(seq - pos, R(1, 1 + seq / 3));
                smp.push_back(b); st.push_back(pos); ln.push_back(len);
                pos += len + R(0, 4);
            }
        const hp_token_map_t m{batch, seq, hiddens[R(0, 6)], R(0, 1), (int32_t)smp.size(), smp.data(), st.data(), ln.data(), nullptr};
        hp_plan p;
        if (hp::build_host_plan(&src, 1, &dst, &m, 1, &p) != HP_OK || p.segments.empty()) continue;
        ++done;
        std::vector<std::vector<int>> image((size_t)p.n_dst_bufs, std::vector<int>((size_t)p.dst_rows_per_buf, 0));
        for (const hp_segment_t &s : p.segments)
            for (int64_t i = 0; i < s.n_rows; ++i) image[s.dst_buf0][s.dst_row0 + i * s.dst_row_stride] = 1;
        const std::vector<hp::Seg> bands = hp::band_runs(p), runs = hp::dst_runs(p, false);
        v = -1;
        CHECK(bands.size() <= runs.size());
        for (v = 0; v < hp::kTileVariants; v += 2) {
            hp::KParams k = hp::kernel_params(p, v, nullptr, nullptr);
            k.band_samples = (uint32_t)p.dst_stride;
            hp::set_division(k.band_samples, k.band_magic, k.band_shift);
            if (k.parts_per_row ? walk<hp::kWholeTiles>(p, bands, k, image) : walk<hp::kRowGroups>(p, bands, k, image)) return 1;
        }
    }
    std::printf("plans %d\n", done);
    return done == plans ? 0 : 2;
}
