// How hp_forward_static takes a plan: reads one from stdin (source tp dp, destination
// tp cp dp zigzag sbh, batch seq hidden f32, images, then sample start length of each)
// and prints its segments and, for each tile size that launches start from, the launches
// that bring the segments (0: tables written into the device's array), whether rows
// are cut, and the bytes of tables.  Built by tests/test_static_tables.py.
#include <cstdio>
#include <vector>

#include "hp_tile.hpp"

int main() {
    hp_layout_t src{}, dst{};
    hp_token_map_t m{};
    src.cp = src.pp = dst.pp = 1;
    if (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d", &src.tp, &src.dp, &dst.tp, &dst.cp, &dst.dp, &dst.cp_split, &dst.row_order, &m.batch,
                   &m.seq, &m.hidden, &m.dtype, &m.n_images) != 12) return 2;
    std::vector<int32_t> sample(m.n_images), start(m.n_images), len(m.n_images);
    for (int32_t k = 0; k < m.n_images; ++k)
        if (std::scanf("%d %d %d", &sample[k], &start[k], &len[k]) != 3) return 2;
    m.img_sample = sample.data(); m.img_start = start.data(); m.img_len = len.data();
    hp_plan p;
    if (hp::build_host_plan(&src, 1, &dst, &m, 1, &p) != HP_OK) return 1;
    std::printf("%zu", p.segments.size());
    for (int v = 0; v < hp::kCutVariants; ++v) {
        const bool cut = hp::cuts_launch(p, 0, v);
        const hp::TreeInfo &t = cut ? p.cut_info[v] : p.tree_info[v];
        const size_t tree = (t.level_off[t.n_levels - 1] + hp::kTreeFanout - t.level_off[0]) * sizeof(uint32_t);
        std::printf(" %zu %d %zu", hp::static_launches(p, tree), (int)cut, (p.segments.size() * sizeof(hp::Seg) + 63) / 64 * 64 + tree);
    }
    std::printf("\n");
    return 0;
}
