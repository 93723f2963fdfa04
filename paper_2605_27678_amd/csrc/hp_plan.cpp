// Host-side plan builder: turns two module grids and one or more token maps
// into the segment tables the gfx950 kernels consume.  Pure C++, no HIP calls.
//
// The step it implements is the one the paper describes for communicator
// construction (Colocated communicator, second paragraph: derive every rank's
// source coordinate, destination coordinate and batch interval from G_u, G_v;
// Non-colocated communicator: both sides construct the same static routing
// pattern) plus the recorded metadata of the reverse transform ("Pipeline
// schedule details", phase 1).  Because the tables list (source run ->
// destination run) pairs, the same table drives forward and backward.
#include "hp_plan.hpp"

#include <algorithm>
#include <cstring>
#include <limits>
#include <new>
#include <numeric>
#include <tuple>

namespace hp {

Options &options() {
    static Options o;
    return o;
}

std::mutex &options_mutex() {
    static std::mutex m;
    return m;
}

int tile_variant_of(int64_t tile_bytes) {
    for (int v = 0; v < kTileVariants; ++v)
        if (tile_bytes == (int64_t)tile_bytes_of(v)) return v;
    return -1;
}

// Dense runs are cut by bytes.  Row-strided ones are cut row by row: a row at
// least one tile long is cut into ceil(row / tile) dense pieces, shorter rows are
// grouped tile / row to a tile.  The kernels use the same formulas.
namespace {
struct TileCount {
    uint64_t row_bytes;
    uint32_t tile_shift, parts, rows_per;           // parts: of a row of at least a tile; rows_per: rows in a tile; both 0 = dense
    TileCount(bool dense, int64_t row, uint32_t tile) : row_bytes((uint64_t)row), tile_shift(10), parts(0), rows_per(0) {
        while ((1u << tile_shift) < tile) ++tile_shift;
        if (dense) return;
        if (row_bytes >= tile) parts = (uint32_t)((row_bytes + tile - 1) >> tile_shift);
        else rows_per = tile / (uint32_t)row_bytes;
    }
    uint64_t operator()(uint64_t n_rows) const {
        if (parts) return n_rows * parts;
        if (!rows_per) return (n_rows * row_bytes + ((1u << tile_shift) - 1)) >> tile_shift;
        if (n_rows <= UINT32_MAX - rows_per) return ((uint32_t)n_rows + rows_per - 1) / rows_per;    // half the time of a division in 64 bits
        return (n_rows + rows_per - 1) / rows_per;
    }
};
}  // namespace

uint64_t tiles_of(uint64_t n_rows, uint64_t pitch_rows, int64_t row_bytes, uint32_t tile) {
    return TileCount(pitch_rows == 1, row_bytes, tile)(n_rows);
}

std::vector<Seg> dst_runs(const hp_plan &p, bool whole) {
    std::vector<Seg> runs;
    if (whole) {                                           // dense, whatever the row order
        for (int64_t buf = 0; buf < p.n_dst_bufs; buf += p.dst_copies)
            for (int64_t row = 0; row < p.dst_rows_per_buf; row += kMaxSegRows) {
                const uint64_t off = (uint64_t)row * (uint64_t)p.row_bytes;
                const int64_t n = std::min<int64_t>(p.dst_rows_per_buf - row, kMaxSegRows);
                runs.push_back(Seg{off, off, (uint32_t)n, 1, (uint16_t)buf, (uint16_t)buf, 0});
            }
        return runs;
    }
    const int64_t stride = p.dst_stride;
    std::vector<size_t> order(p.segments.size());
    std::iota(order.begin(), order.end(), (size_t)0);
    auto place = [&](size_t i) {                           // buffer, column, position in the column
        const hp_segment_t &s = p.segments[i];
        return std::make_tuple((int64_t)s.dst_buf0, s.dst_row0 % stride, s.dst_row0 / stride);
    };
    std::sort(order.begin(), order.end(), [&](size_t a, size_t b) { return place(a) < place(b); });
    const int64_t column = p.dst_rows_per_buf / stride;
    size_t at = 0;
    for (int64_t buf = 0; buf < p.n_dst_bufs; buf += p.dst_copies)
        for (int64_t col = 0; col < stride; ++col) {
            int64_t done = 0;                              // rows of this column that have a run
            auto add = [&](int64_t rows, uint32_t image) {
                if (rows <= 0) return;
                if (done > 0 && runs.back().src_copies == image && runs.back().n_rows + rows <= (int64_t)kMaxSegRows) {
                    runs.back().n_rows += (uint32_t)rows;
                    done += rows;
                }
                else while (rows > 0) {
                    const int64_t n = std::min<int64_t>(rows, kMaxSegRows);
                    const uint64_t off = (uint64_t)(done * stride + col) * (uint64_t)p.row_bytes;
                    runs.push_back(Seg{off, off, (uint32_t)n, (uint32_t)stride, (uint16_t)buf, (uint16_t)buf, image});
                    done += n;
                    rows -= n;
                }
            };
            for (; at < order.size(); ++at) {
                const hp_segment_t &s = p.segments[order[at]];
                if (s.dst_buf0 != buf || s.dst_row0 % stride != col) break;
                add(s.dst_row0 / stride - done, 0);
                add(s.n_rows, 1);
            }
            add(column - done, 0);
        }
    return runs;
}

std::vector<Seg> band_runs(const hp_plan &p) {
    struct Turn { int64_t buf, pos; uint32_t sample; };    // where a sample (a bit) goes from text to image or back
    const int64_t samples = p.dst_stride, positions = p.dst_rows_per_buf / samples;
    std::vector<Turn> turns;
    turns.reserve(2 * p.segments.size());
    for (const hp_segment_t &s : p.segments) {
        const uint32_t bit = 1u << (s.dst_row0 % samples);
        turns.push_back(Turn{s.dst_buf0, s.dst_row0 / samples, bit});
        turns.push_back(Turn{s.dst_buf0, s.dst_row0 / samples + s.n_rows, bit});
    }
    std::sort(turns.begin(), turns.end(), [](const Turn &a, const Turn &b) {
        return a.buf != b.buf ? a.buf < b.buf : a.pos < b.pos;
    });
    std::vector<Seg> runs;
    size_t at = 0;
    for (int64_t buf = 0; buf < p.n_dst_bufs; buf += p.dst_copies) {
        int64_t done = 0;                                  // positions that have a run
        uint32_t images = 0;
        auto add = [&](int64_t end) {
            while (done < end) {                           // a band's rows stay below 2^31, as the kernels' division wants them
                const int64_t n = std::min<int64_t>(end - done, INT32_MAX / samples);
                const uint64_t off = (uint64_t)(done * samples) * (uint64_t)p.row_bytes;
                runs.push_back(Seg{off, off, (uint32_t)(n * samples), 1, (uint16_t)buf, (uint16_t)buf, images});
                done += n;
            }
        };
        while (at < turns.size() && turns[at].buf == buf) {
            const int64_t pos = turns[at].pos;
            uint32_t next = images;
            for (; at < turns.size() && turns[at].buf == buf && turns[at].pos == pos; ++at) next ^= turns[at].sample;
            if (next != images) add(pos);                  // else one image ends where the next begins
            images = next;
        }
        add(positions);
    }
    return runs;
}

namespace {

// Position of one fused-sequence token on the destination side.
struct DstPos {
    int32_t buf0;   // first buffer that holds it
    int64_t s_loc;  // position inside that buffer's local sequence
    int64_t run;    // tokens from here on that stay consecutive in this buffer
};

// Walks the destination grid's definition for sample-local position s of a
// sample owned by dp rank `dp`.
struct DstWalker {
    int32_t tp, cp, mode, split;
    int64_t per_cp;   // positions per cp rank
    int64_t chunk;    // zigzag chunk length
    int64_t piece;    // positions per buffer (per_cp, or per_cp/tp when sharded)

    DstWalker(const hp_layout_t &g, int64_t seq)
        : tp(g.tp), cp(g.cp), mode(g.tp_mode), split(g.cp_split) {
        per_cp = seq / cp;
        chunk = (split == HP_CP_ZIGZAG) ? seq / (2 * (int64_t)cp) : per_cp;
        piece = (mode == HP_TP_SEQ_SHARD) ? per_cp / tp : per_cp;
    }

    DstPos at(int32_t dp, int64_t s) const {
        int64_t q = s / chunk, r = s - q * chunk;
        int32_t c;
        int64_t in_cp;
        if (split == HP_CP_ZIGZAG) {
            // chunks 0..C-1 are the first halves of ranks 0..C-1, chunks C..2C-1
            // are the second halves of ranks C-1..0
            if (q < cp) { c = (int32_t)q; in_cp = r; }
            else        { c = (int32_t)(2 * (int64_t)cp - 1 - q); in_cp = chunk + r; }
        } else {
            c = (int32_t)q; in_cp = r;
        }
        DstPos p;
        p.run = chunk - r;
        int32_t slice = c + cp * dp;
        if (mode == HP_TP_SEQ_SHARD) {
            int64_t t = in_cp / piece;
            p.s_loc = in_cp - t * piece;
            p.run = std::min<int64_t>(p.run, piece - p.s_loc);
            p.buf0 = (int32_t)t + tp * slice;
        } else {
            p.s_loc = in_cp;
            p.buf0 = tp * slice;
        }
        return p;
    }
};

int validate(const hp_layout_t *src, const hp_layout_t *dst, const hp_token_map_t *m) {
    if (!src || !dst || !m) return HP_EINVAL;
    for (const hp_layout_t *g : {src, dst}) {
        if (g->tp < 1 || g->cp < 1 || g->dp < 1 || g->pp < 1 || g->rank_offset < 0) return HP_EINVAL;
        if (g->tp_mode != HP_TP_REPLICATE && g->tp_mode != HP_TP_SEQ_SHARD) return HP_EINVAL;
        if (g->cp_split != HP_CP_CONTIGUOUS && g->cp_split != HP_CP_ZIGZAG) return HP_EINVAL;
        if (g->row_order != HP_ROW_BSH && g->row_order != HP_ROW_SBH) return HP_EINVAL;
    }
    if (m->batch < 1 || m->seq < 1 || m->hidden < 1 || m->n_images < 0) return HP_EINVAL;
    if (m->dtype != HP_BF16 && m->dtype != HP_F32) return HP_EINVAL;
    if (m->n_images > 0 && (!m->img_sample || !m->img_start || !m->img_len)) return HP_EINVAL;

    // the encoder side has no context parallelism and plain replicated TP
    if (src->cp != 1 || src->tp_mode || src->cp_split || src->row_order) return HP_ELAYOUT;
    if (m->batch % dst->dp) return HP_ELAYOUT;
    if (m->seq % dst->cp) return HP_ELAYOUT;
    if (dst->cp_split == HP_CP_ZIGZAG && m->seq % (2 * (int64_t)dst->cp)) return HP_ELAYOUT;
    if (dst->tp_mode == HP_TP_SEQ_SHARD && (m->seq / dst->cp) % dst->tp) return HP_ELAYOUT;
    if ((int64_t)src->tp * src->dp + (int64_t)dst->tp * dst->cp * dst->dp > HP_MAX_BUFFERS) return HP_ELAYOUT;
    if (dst->tp_mode == HP_TP_REPLICATE && dst->tp > HP_MAX_TP) return HP_ELAYOUT;

    // spans
    int32_t prev_sample = 0, prev_dp = 0;
    for (int32_t k = 0; k < m->n_images; ++k) {
        int32_t b = m->img_sample[k];
        int64_t s = m->img_start[k], n = m->img_len[k];
        if (b < 0 || b >= m->batch || b < prev_sample) return HP_EMAP;
        if (s < 0 || n < 1 || s + n > m->seq) return HP_EMAP;
        prev_sample = b;
        if (m->img_src_dp) {
            int32_t d = m->img_src_dp[k];
            if (d < 0 || d >= src->dp || d < prev_dp) return HP_EMAP;
            prev_dp = d;
        }
    }
    // overlap inside a sample: order each sample's spans by start
    std::vector<int32_t> order(m->n_images);
    std::iota(order.begin(), order.end(), 0);
    std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        if (m->img_sample[a] != m->img_sample[b]) return m->img_sample[a] < m->img_sample[b];
        return m->img_start[a] < m->img_start[b];
    });
    for (size_t i = 1; i < order.size(); ++i) {
        int32_t a = order[i - 1], b = order[i];
        if (m->img_sample[a] == m->img_sample[b] &&
            (int64_t)m->img_start[a] + m->img_len[a] > m->img_start[b])
            return HP_EMAP;
    }
    return HP_OK;
}

int make_tables(hp_plan *p) {
    const size_t n = p->segments.size();
    p->dsegs.resize(n);
    for (size_t i = 0; i < n; ++i) {
        const hp_segment_t &s = p->segments[i];
        Seg &d = p->dsegs[i];
        d.src_off = (uint64_t)s.src_row0 * p->row_bytes;
        d.dst_off = (uint64_t)s.dst_row0 * p->row_bytes;
        if (s.n_rows < 1 || s.n_rows > (int64_t)kMaxSegRows || s.dst_row_stride < 1 ||
            s.dst_row_stride > (int64_t)UINT32_MAX || s.src_buf > UINT16_MAX || s.dst_buf0 > UINT16_MAX)
            return HP_ELAYOUT;                                // would not fit the descriptor's fields
        d.n_rows = (uint32_t)s.n_rows;
        d.src_copies = (uint32_t)p->seg_copies[i];
        d.pitch_rows = (uint32_t)s.dst_row_stride;
        d.src_buf = (uint16_t)s.src_buf;
        d.dst_buf0 = (uint16_t)s.dst_buf0;
    }
    p->first_tile.resize((size_t)kTileVariants * (n + 1));
    // The first tile of every segment; false if there are more than a grid may have.
    auto count = [&](const TileCount &tiles, uint32_t *keys, uint32_t &all) {
        uint64_t acc = 0;
        for (size_t i = 0; i < n; ++i) {
            keys[i] = (uint32_t)acc;
            acc += tiles((uint64_t)p->segments[i].n_rows);
            if (acc > 0x7fffffffull) return false;
        }
        all = (uint32_t)acc;
        return true;
    };
    for (int v = 0; v < kTileVariants; ++v) {
        uint32_t *row = p->first_tile.data() + (size_t)v * (n + 1);
        if (!count(TileCount(p->dst_stride == 1, p->row_bytes, tile_bytes_of(v)), row, row[n])) return HP_ELAYOUT;
    }
    // Which tile sizes can be cut across the ends of rows.
    const int64_t row_bytes = p->row_bytes;
    bool cut = n > 0 && p->dst_stride > 1 && row_bytes <= kMaxCutRow && (row_bytes % 128 == 0 || row_bytes >= kMinPaddedRow);
    for (size_t i = 0; i < n && cut; ++i) cut = p->segments[i].n_rows * cut_row_lines(row_bytes) <= INT32_MAX;    // the kernels divide lines in 31 bits
    // 16-ary search trees over the keys of each variant.  Plans are made at step rate, and this and the counts are most
    // of it: each level is written where it stays.
    const size_t padded = (n + kTreeFanout - 1) / kTreeFanout * kTreeFanout;
    p->tree.clear();
    p->tree.reserve((kTileVariants + (cut ? kCutVariants : 0)) * (padded + padded / (kTreeFanout - 1) + kMaxTreeLevels * kTreeFanout));
    auto add_tree = [&](const uint32_t *keys, TreeInfo &ti) -> int {
        ti.n_levels = 0;
        size_t below = n;                                   // keys of the level
        for (;; below = (below + kTreeFanout - 1) / kTreeFanout) {
            if (ti.n_levels == (uint32_t)kMaxTreeLevels) return HP_ELAYOUT;
            const size_t at = p->tree.size(), under = ti.n_levels ? ti.level_off[ti.n_levels - 1] : 0;
            p->tree.resize(at + (below + kTreeFanout - 1) / kTreeFanout * kTreeFanout, 0xffffffffu);
            uint32_t *level = p->tree.data() + at;
            if (ti.n_levels == 0) std::memcpy(level, keys, n * sizeof(uint32_t));
            else for (size_t j = 0; j < below; ++j) level[j] = p->tree[under + j * kTreeFanout];
            ti.level_off[ti.n_levels++] = (uint32_t)at;
            if (below <= (size_t)kTreeFanout) return HP_OK;
        }
    };
    int rc = HP_OK;
    for (int v = 0; v < kTileVariants && n > 0 && rc == HP_OK; ++v)
        rc = add_tree(p->first_tile.data() + (size_t)v * (n + 1), p->tree_info[v]);
    std::vector<uint32_t> keys(cut ? n : 0);
    for (int v = 0; v < kTileVariants; ++v) {
        p->cut_tiles[v] = 0;
        const int64_t tile = tile_bytes_of(v);
        if (rc != HP_OK || !cut || v >= kCutVariants || (row_bytes % 128 == 0 && (row_bytes % tile == 0 || tile % row_bytes == 0))) continue;
        if (!count(TileCount(true, 128 * cut_row_lines(row_bytes), (uint32_t)tile), keys.data(), p->cut_tiles[v])) continue;
        rc = add_tree(keys.data(), p->cut_info[v]);
    }
    return rc;
}

// The share of a tile that row-strided rows fill where they are cut one by one, or as many as fit lie in it whole.
double row_share(int64_t row, int64_t tile) {
    return row >= tile ? (double)row / (double)((row + tile - 1) / tile * tile) : (double)(tile / row * row) / (double)tile;
}
// Whether rows that are not whole lines fill tiles of lines enough better: see cuts_launch.
// Groups of shorter rows store between 64-byte pieces, padded ones do not, and may fill less; but not in tiles of 1 KiB, whose
// few chunks hide that: forward 0.91-1.08 at 60 MB to 2.5 GB, 0.98 in the middle (rows of 600 bytes to three and four
// copies, 120 MB, 0.88-0.97).
bool padding_pays(const hp_plan &p, int variant, int direction) {
    const int64_t row = p.row_bytes, tile = tile_bytes_of(variant);
    if (direction == 0 && tile == 1024 && row < tile) return false;
    const double more = row >= tile ? 0.03 : direction != 0 ? -0.12 : tile == 8192 ? -0.25 : -0.15;
    return row % 128 && p.cut_tiles[variant] && (double)row / (double)(128 * cut_row_lines(row)) >= row_share(row, tile) + more;
}
// Row-strided rows that launches in small tiles can cut by bytes; those of 2 KiB and more want what dense launches want.
bool cut_rows(const hp_plan &p) { return p.row_bytes % 128 == 0 && (p.cut_tiles[0] || p.cut_tiles[1]); }
bool like_dense(const hp_plan &p) { return p.row_bytes >= 2048 && p.row_bytes % 128 == 0 && p.cut_tiles[0]; }

// Forward to eight copies in short rows, between what tiles of 1 KiB and cutting suit: 0.93-0.97 with either.
bool eight_short(const hp_plan &p, double fwd_bytes) {
    return p.dst_stride > 1 && p.dst_copies == 8 && p.row_bytes < 1536 && fwd_bytes >= 450e6 && fwd_bytes < 1500e6;
}

// Whether all tiles of 1 KiB but a run's last are whole.
bool even_tiles(const hp_plan &p) { return p.dst_stride == 1 || p.row_bytes % 1024 == 0 || like_dense(p); }

// The shapes of launches whose size calls for others than the replica counts
// alone.  Each line was measured against the shape that it replaces in the
// sequence a program runs (forward, backward, forward, ...; forward, accumulate,
// ... - a shape that leaves dirty lines behind is paid for by the next launch,
// and ranks wrongly when it is timed alone) and on the same buffers (two sets
// differ by 2 % and now and then by 10), in both element types, with rows of
// 0.5 to 24 KiB, images of 16 to 4096 rows, both row orders and launches of 8 MB to
// 4.5 GB; the figures are the direction's gain over that range, and after the
// semicolon what it would be where the line has ended.  Copy
// counts measured: 1 to 16 with one source copy; 1 to 8 and 12 with two.
// Launches of up to about 400 MB find part of
// their buffers in the 256 MB memory-side cache and want more waves; replica
// counts without a kernel of their own (all but 1, 2, 3, 4 and 8) wait for their
// groups of four loads and want more of them in flight; the more copies there
// are to write, the fewer waves keep a compute unit's 40 to 50 KB on their way; and
// small tiles want segments and rows that fill them.
void by_size(const hp_plan *p, Launch &f, Launch &b, Launch &a) {
    constexpr int K1 = 0, K2 = 1, K4 = 2, K8 = 3;            // tiles of 1, 2, 4 and 8 KiB
    const int c = p->dst_copies, s = p->src_copies;
    const bool between = c != 1 && c != 2 && c != 4 && c != 8;                  // 3, 5 to 7, 9 to 16 copies
    const bool f32 = p->elem_bytes == 4, dense = p->dst_stride == 1 || like_dense(*p);
    // A row-strided row is cut into tiles from its start: whether it fills what it is cut into, and that in whole lanes.
    const int64_t row = p->row_bytes;
    const bool full = dense || cut_rows(*p) || (row >= 2048 && padding_pays(*p, 0, 0));       // tiles of 1 KiB are whole, or as full as larger ones at least
    auto fills = [&](int64_t tile) { return dense || 20 * row >= 17 * ((row + tile - 1) / tile * tile); };
    const bool filled = fills(1024) && (dense || row % 16 == 0), even = even_tiles(*p);
    const size_t segs = p->segments.size();
    constexpr double MB = 1e6;
    auto set = [](Launch &L, int tile, int block, int cap) { L = Launch{tile, block, cap, L.nontemporal}; };
    auto in = [](double bytes, double from, double to) { return bytes >= from * MB && bytes < to * MB; };

    const double fwd = (1.0 + c) * (double)p->n_rows * (double)p->row_bytes;
    // Rows of three and a half KiB and a little more leave as much of tiles of 1 KiB empty as of 2 KiB.  Forward in the smaller
    // ones, where they are not cut: 0.87-0.97 to four copies, 0.94-0.98 to twelve and more, 0.93-0.99 to eight and ten up to
    // 200 MB (1.02-1.09 above).
    const bool halves = p->dst_stride > 1 && row > 2048 && row < 4096 && row_share(row, 1024) < 0.95 && row_share(row, 1024) <= row_share(row, 2048) &&
                        !cuts_launch(*p, 0, K1) && (c < 8 || c >= 12 || fwd < 200 * MB);
    if (c == 1 && fwd >= 200 * MB && segs <= 256) {
        if (fwd < 400 * MB || !dense) set(f, K4, 128, 24);                      // 0.99-1.03; more segments 0.98-1.03
        else set(f, K2, 64, 20);                                                // 1.003-1.006 of 4 KiB x 128; [S,B,H] 0.92-0.98
    }
    else if (c == 2 && in(fwd, 40, 290)) set(f, K8, 256, 16);                   // 0.98-1.13; 300 MB: 0.96-1.00
    else if (c == 2 && fwd >= 300 * MB && filled) {
        if (segs <= 256) set(f, K1, 64, 20);                                    // 1.01-1.04 to 1.2 GB, 1.01-1.02 to 15 GB; else 0.93-1.02
        else if (segs <= 1024 && fwd >= 1500 * MB) set(f, K1, 64, 24);          // 1.01-1.03; smaller launches and more segments 0.97-1.02
    }
    else if (c == 3 && in(fwd, 40, 1000)) {
        if (segs <= 128 && (filled || row < 1024)) set(f, K1, 64, fwd < 200 * MB ? 10 : 16);   // 1.00-1.14; more segments 0.94-1.0, rows of 1280 and 3088 bytes 0.87-0.99
    }
    else if (c == 4 && in(fwd, 8, 180)) {
        if (segs <= 256 && (filled || row < 1024)) set(f, K1, 64, 8);           // 0.99-1.15; more segments 0.96-1.02, rows of 1280 bytes 0.92, 450 MB 0.87-0.91
    }
    else if (c == 4 && in(fwd, 180, 1000)) {
        if (segs <= (fwd < 900 * MB ? 512 : 256) && row > 2048 && !halves) set(f, K1, 64, fwd < 450 * MB ? 12 : 14);   // 1.00-1.13; 1 to 4 GB 0.99-1.03, rows of 1 and 2 KiB 0.98-1.03, two thousand segments 0.91-1.0
    }
    else if (c >= 5 && c <= 7 && in(fwd, 40, 450)) {
        if (c > 5 || segs <= 16) set(f, K1, 64, 10);                            // 0.96-1.20; 20 MB 0.89-1.06, five copies and more segments 0.87-1.03
    }
    else if (c >= 5 && c <= 7 && fwd >= 450 * MB) {
        if (segs <= (c == 5 ? 256 : 1024) && (filled || row < 2048)) set(f, K1, 64, 14);   // 1.00-1.15; more segments 0.97-1.02, rows of 3088 and 8186 bytes 0.94-0.99
    }
    else if (c == 8 && full && !halves && in(fwd, 40, 450)) set(f, K1, 64, 5);            // 0.99-1.25; [S,B,H] order, four and two samples, cut or not, 0.96-1.25
    else if (c == 8 && full && in(fwd, 450, 5000) && !eight_short(*p, fwd)) {
        if (segs <= 256) set(f, K1, 64, fwd < 700 * MB ? 5 : 8);                // 1.00-1.06; more segments 0.98-1.02, 7.2 GB 0.99; [S,B,H] 0.94-1.24
    }
    else if (c >= 10 && c <= 12 && full && !halves && in(fwd, 100, c == 12 ? 450 : 600)) set(f, K1, 64, 5);   // 0.96-1.28; ten copies, 700 MB 0.98-1.0, 1.1 GB 0.85; [S,B,H] 0.95-1.20
    else if (c == 12 && full && in(fwd, 450, 1200)) {
        if (segs <= 256) set(f, K1, 64, fwd < 1000 * MB ? 3 : 4);               // 1.02-1.12; 1.2 GB 0.93-0.99
    }
    else if (c >= 13 && c <= 15 && full && !halves && in(fwd, 100, 1200)) set(f, K1, 64, 4);  // 0.98-1.10; 1.4 GB 0.94-1.03
    else if (c == 16 && full && !halves && in(fwd, 100, 1500)) set(f, K1, 64, 3);         // 1.01-1.11, paced; 1.7 GB 0.91-0.99; [S,B,H], not paced, 0.97-1.12
    else if (c >= 13 && full && fwd >= 1200 * MB) set(f, K2, 64, 3);   // 0.99-1.03 to 4 GB

    // With few copies a workgroup moves little for each search, and the depth of the tree (16 segments a level) decides.
    const double bwd = (double)p->bwd_bytes;
    if (c == 1 && s == 1 && in(bwd, 25, 200)) {
        if (segs <= 16) set(b, K1, 64, 28);                                     // 1.01-1.09; more segments 0.73-0.86
    }
    else if (c == 1 && s == 1 && bwd >= 200 * MB) {
        if (segs <= 256) set(b, K4, 128, 24);                                   // 0.99-1.04; more segments 0.95-1.00
    }
    else if (c == 2 && s == 1 && in(bwd, 80, 290)) {
        if (segs <= 16) set(b, K8, 256, 24);                                    // 0.99-1.06; more segments 0.95-1.02, 40 MB 0.97-1.05
    }
    else if (c == 2 && s == 1 && bwd >= 400 * MB && even) {
        if (segs <= 16) set(b, K1, 64, 28);                                     // 1.00-1.02
        else if (segs <= 4096) set(b, K1, 64, segs <= 1024 ? 24 : 28);          // paced: 1.01-1.04 of cap 30
    }
    else if (c == 2 && s > 1 && bwd >= 40 * MB) set(b, K1, 64, 20);             // 1.05-1.09; 27 MB: 0.95-1.02
    else if (c == 4 && s == 1 && in(bwd, 35, segs <= 16 ? 360 : 220)) set(b, K1, 64, 24);   // 1.02-1.14; more segments from 240 MB 0.95-1.04
    else if (between && c < 8 && bwd >= (c <= 5 ? 16 : 30) * MB &&              // 3 copies 1.03-1.35, 5 to 7 0.98-1.28
             !(f32 && (s > 1 ? bwd >= 600 * MB : c == 7 && bwd >= 500 * MB)))   // there 0.97-1.02 and 0.95-1.02
    {
        int cap = c <= 5 && s == 1 ? 28 : 24;
        if (c == 3 && s == 1 && bwd >= 450 * MB && even) cap = segs <= 4096 ? 20 : 24;   // paced: 1.01-1.03 of cap 28
        else if (c == 5 && bwd >= 450 * MB && filled) cap = bwd < 800 * MB ? 20 : 16;   // 1.00-1.02
        else if (c == 6 && bwd >= 450 * MB && filled) cap = 16;                 // 1.01-1.02
        set(b, K1, 64, cap);
    }
    // half a dozen to a dozen waves of eight and more copies have to have whole tiles: [S,B,H] rows that leave them partly empty lose 2-13 % here (2560 bytes, cut from 400 MB on, 0.96-1.04)
    else if (c == 8 && bwd >= 1500 * MB && (dense || row < 4096 || fills(4096))) set(b, K4, 64, 5);   // 1.01-1.06, to two source copies 1.05-1.11
    else if (c == 8 && bwd >= 40 * MB && filled) set(b, K1, 64, bwd < 450 * MB ? 12 : 11);   // 1.00-1.03
    else if (c > 12 && p->dst_stride == 1 && in(bwd, 40, 250)) set(b, K1, 64, 12);           // 1.02-1.07; 350 MB 0.97-1.00, [S,B,H] order 0.85-1.0
    else if (c > 8 && bwd >= 600 * MB && filled) set(b, K1, 64, 10);            // 1.02-1.06
    else if (c > 8 && !f32 && in(bwd, 100, 250)) set(b, K4, 128, 24);           // 0.98-1.14; binary32: 0.97-1.00, 300 MB: 0.94-1.01

    const double acc = (double)p->bwd_accum_bytes;
    if (acc < 1 * MB) return;                                                   // a few tiles: nothing to choose
    const bool whole = dense || row >= 4096;                 // tiles of 1 KiB are nearly all whole
    // In 4 KiB row-strided rows want what dense ones want where they are cut there: rows of 3712, 3968 and 7552 bytes, which
    // are not, 0.87-0.95 with the wave cap of dense launches (one to three copies, and eight).
    const bool dense4 = p->dst_stride == 1 || (dense && cuts_launch(*p, 2, K4));
    if (f32) {
        // More waves make these launches faster and the forward after them slower by as much: only the middle sizes gain,
        // and none with several source copies (0.77-1.05).
        const bool gains = c <= 5 ? in(acc, 90, 200)                            // 0.99-1.11; 48 MB: 0.93-1.02, 400 MB: 0.74-1.04
                           : c < 8 ? acc < 350 * MB                             // 1.01-1.48; 680 MB: 0.81-0.97
                           : c == 8 ? dense && in(acc, 150, 400)                // 1.00-1.05; 670 MB: 0.84-0.89
                                    : acc < 300 * MB;                           // 1.02-1.30; 1.6 GB: 0.87-0.97
        if (s == 1 && gains) set(a, K1, 64, 24);
        else if (c <= 2 && s == 1 && acc >= 1500 * MB && (dense || row % 4096 == 0))
            set(a, K4, 64, 8);                                                  // 1.02-1.06; 450 MB: 0.97-1.01, [S,B,H] rows of 6 KiB 0.93
    } else if (s > 1) {
        // few waves want whole tiles: pieces of row-strided rows under 4 KiB 0.96-1.01 with the smaller caps, 1.02-1.13 with 16
        if (acc < 200 * MB || (between && !whole)) set(a, K1, 64, 16);          // 1.04-1.44
        else if (between) set(a, K1, 64, c > 8 && acc >= 400 * MB ? 10 : acc < 1000 * MB ? 16 : 13);   // 0.99-1.04; cap 16 to the end 0.98-1.00
        else if (whole && (c == 4 || c == 8)) set(a, K1, 64, c == 4 ? 13 : 8);  // 0.98-1.09; else 0.98-1.04
    } else if (acc < 400 * MB) {
        if (c == 2 && acc >= 350 * MB && filled) set(a, K1, 64, 16);              // 1.02
        else if (c >= 3 && c <= 7 && acc >= 250 * MB) set(a, K1, 64, c == 3 ? 20 : c == 4 ? 14 : 16);   // 1.01-1.03; 200 MB 0.99-1.01
        else if (c == 2 ? acc < 280 * MB : c <= 5) set(a, K4, 256, dense4 ? 24 : 0);         // 0.97-1.48; two copies, 300 MB: 0.99-1.02
        else if (c >= 5 && c < 8) set(a, K1, 64, 24);                           // 1.10-1.63
        else if (c == 8 && dense4 && in(acc, 50, 350)) set(a, K4, 256, 16);      // 1.01-1.11; 27 MB 0.96, 400 MB 0.99, [S,B,H] 0.96-1.07
        else if (c > 8) set(a, K1, 64, c <= 10 || acc < 150 * MB ? 20 : 12);    // 1.21-1.71, cap 12 1.00-1.02 on top; 9 copies 0.99
    } else if (c == 1 || (between && !whole)) {
        set(a, K1, 64, c < 8 ? 20 : 16);                                        // 1.00-1.02, pieces of short rows 1.02-1.15
    } else if (c == 2) {
        if (filled) set(a, K1, 64, 16);                                           // 1.01-1.02, from 2 GB on 1.00; [S,B,H] rows of 6 KiB 1.15, not of whole lanes 0.94-0.98
    } else if (c == 3) {
        if (acc < 1500 * MB) set(a, K1, 64, 20);                                // 1.01-1.02
        else set(a, K2, 64, 11);                                                // 1.01-1.02
    } else if (c == 4) {
        set(a, K2, 64, 8);                                                      // 1.01-1.02
    } else if (c == 5) {
        set(a, K1, 64, acc < 1000 * MB ? 16 : 14);                              // 1.02-1.26; cap 20 to the end 0.97-0.99
    } else if (c < 8) {
        set(a, K1, 64, acc < 600 * MB ? 16 : 13);                               // 1.02-1.26; cap 16 to the end 0.99-1.02
    } else if (c > 8) {
        set(a, K1, 64, c < 13 ? 12 : 11);                                       // 1.20-1.37; cap 10 0.99-1.00
    } else if (acc >= 450 * MB) {
        set(a, K1, 64, 10);                                                     // eight copies: 1.02-1.05
    }
}

// HIP refuses a grid of 2^32 work-items or more: 64 GiB in tiles of 1 KiB, one
// wave each.  Such a launch takes the next larger tiles.
void keep_grid(const hp_plan *p, Launch &L) {
    constexpr uint64_t kItems = (uint64_t)1 << 32;
    const uint64_t most = std::max<uint64_t>((uint64_t)(p->n_rows * p->row_bytes) >> 10, (uint64_t)p->n_rows);
    if ((most + p->segments.size()) * (uint64_t)L.block < kItems) return;
    for (; L.tile_variant + 1 < kTileVariants; ++L.tile_variant) {
        uint64_t tiles = 0;
        for (const hp_segment_t &s : p->segments)
            tiles += tiles_of((uint64_t)s.n_rows, (uint64_t)s.dst_row_stride, p->row_bytes, tile_bytes_of(L.tile_variant));
        if (tiles * (uint64_t)L.block < kItems) return;
    }
}

// Launch shapes for a new plan.  Both kernels are fastest when roughly 100 KB
// of traffic per compute unit is in flight, so the resident-wave cap that suits
// a plan falls as the number of buffers a row's traffic spreads over rises:
// 1 + dst_copies for forward, dst_copies + src_copies for backward.  The table
// is what the measured search (hp_plan_tune) picks most often per replica count
// on the five workloads and their sequence-sharded variants; by_size puts others
// in their place where the launch's size calls for it; an option that is not
// HP_AUTO overrides its field.
void default_launches(hp_plan *p) {
    Options o;
    {
        std::lock_guard<std::mutex> lk(options_mutex());
        o = options();
    }
    const int c = p->dst_copies, s = p->src_copies;
    Launch f{1, 64, c <= 1 ? 24 : c <= 4 ? 12 : c <= 7 ? 8 : 5, 2};                          // 2 KiB tiles
    if (c == 2) f = Launch{2, 256, 28, 2};      // two copies: 4 KiB tiles, 256 lanes, where by_size has no other (from 300 MB on that is many segments and rows that fill small tiles badly)
    Launch b = c + s <= 2 ? Launch{1, 64, 30, 3} : c + s == 3 ? Launch{0, 64, 30, 3} : Launch{0, 64, 16, 3};
    // accumulating backward: the binary32 accumulators are read and written, 2 * 4 / elem_bytes row sizes per copy;
    // caps as the measured search finds them for 6, 8 and 16 streams (two, four and eight copies; the last from two source copies)
    const int acc_streams = c + s * 8 / p->elem_bytes;
    Launch a{1, 64, acc_streams <= 4 ? 16 : acc_streams <= 6 ? 13 : acc_streams <= 8 ? 11 : acc_streams <= 12 ? 9 : 7, 3};
    by_size(p, f, b, a);
    for (Launch *L : {&f, &b, &a}) keep_grid(p, *L);
    auto apply = [](Launch &L, int64_t tile, int64_t block, int64_t waves, int64_t nt) {
        if (tile > 0) L.tile_variant = tile_variant_of(tile);
        if (block > 0) L.block = (int32_t)block;
        if (waves >= 0) L.waves_per_cu = (int32_t)waves;
        L.nontemporal = (int32_t)nt;
    };
    apply(f, o.tile_bytes_fwd, o.block_threads_fwd, o.waves_per_cu_fwd, o.nontemporal_fwd);
    apply(b, o.tile_bytes_bwd, o.block_threads_bwd, o.waves_per_cu_bwd, o.nontemporal_bwd);
    apply(a, o.tile_bytes_bwd > 0 ? std::max<int64_t>(o.tile_bytes_bwd, 4096) : -1, o.block_threads_bwd,
          o.waves_per_cu_bwd, o.nontemporal_bwd);
    p->fwd = f;
    p->bwd = b;
    p->acc = a;
}

// No two spans of one microbatch may overlap, whichever edge they belong to.
int check_cross_edge_overlap(const hp_token_map_t *maps, int32_t n_edges, int32_t n_maps) {
    struct Span { int32_t b; int64_t s, e; };
    std::vector<Span> spans;
    for (int32_t mi = 0; mi < n_maps; ++mi) {
        spans.clear();
        for (int32_t e = 0; e < n_edges; ++e) {
            const hp_token_map_t &m = maps[(size_t)e * n_maps + mi];
            for (int32_t k = 0; k < m.n_images; ++k)
                spans.push_back(Span{m.img_sample[k], m.img_start[k], (int64_t)m.img_start[k] + m.img_len[k]});
        }
        std::sort(spans.begin(), spans.end(), [](const Span &x, const Span &y) {
            return x.b != y.b ? x.b < y.b : x.s < y.s;
        });
        for (size_t i = 1; i < spans.size(); ++i)
            if (spans[i].b == spans[i - 1].b && spans[i].s < spans[i - 1].e) return HP_EMAP;
    }
    return HP_OK;
}

}  // namespace

// How many: few enough that the scalar unit still keeps ahead of memory; past that a
// launch takes longer with every round.  Measured on the same buffers in turn, 0 to 28
// rounds, over 0.45 to 4.5 GB, both element types, whole and ragged rows.  The gain is
// over no pacing, either at its best cap, by the levels of the search tree (which take
// the place of some rounds); in brackets what is left of it three rounds either way.
//   backward, two copies     -, 1.02 (0.99-1.01), 1.01 (1.00)
//             three          1.02 (1.01), 1.02 (1.00-1.01), 1.02 (1.01)
//             four           1.02 (1.01), 1.02 (1.01), 1.02 (1.01)
//             six, 0.8 GB on 1.01-1.02 (1.01), 1.01 (1.01), -
//   forward, sixteen, 0.2 to 1.5 GB 1.03 (1.02), 1.03 (1.02), 1.01 (1.00)
// Against the kernels whose search was slower and paced them by itself the paced ones
// are at 1.00-1.01 (two copies, two levels), 1.13 (three), 1.00-1.03 (three copies), 1.01-1.03
// (four), 1.05 (six).  Elsewhere - smaller launches, other counts, four levels, accumulating,
// forward to 13 to 15 copies - pacing gains 1 % at most or loses.  Where row-strided rows
// leave tiles partly empty it costs up to 13 %.
int pace_rounds(const hp_plan &p, int direction, const Launch &L) {
    static const uint8_t two[] = {0, 7, 3, 0}, three[] = {18, 13, 8, 0}, four[] = {21, 17, 12, 0}, six[] = {25, 22, 0, 0}, sixteen[] = {12, 9, 3, 0};
    if (L.tile_variant != 0 || L.block != 64 || p.src_copies != 1 || !even_tiles(p) || p.segments.empty()) return 0;
    const int c = p.dst_copies, level = (int)p.tree_info[0].n_levels - 1;
    if (direction == 0) {
        const double bytes = (1.0 + c) * (double)p.n_rows * (double)p.row_bytes;
        return c == 16 && p.dst_stride == 1 && bytes >= 200e6 && bytes < 1.5e9 ? sixteen[level] : 0;
    }
    const double bytes = (double)p.bwd_bytes;
    if (direction != 1 || bytes < 400e6) return 0;
    return c == 2 ? two[level] : c == 3 && bytes >= 450e6 ? three[level] : c == 4 ? four[level] : c == 6 && bytes >= 800e6 ? six[level] : 0;
}

// Where rows are not whole lines, a tile's ends lie on lines of one side only, and on the
// other two tiles share the lines at their ends.  Stores lose more by that than loads: backward, tiles on lines of
// the source that is written instead of the copies that are read (rows of 2008 to 16816 bytes, 0.1 to 2 GB,
// the same buffers in turn) one copy 1.02-1.09 (two 0.99, four 0.93-0.95); to two source copies from one 1.08-1.28,
// from two 1.04-1.14, from three 1.02-1.13, from four 1.00-1.06; to three and four from twice as many 1.02-1.07;
// from four and more in 40 MB 0.94-1.0.  Accumulating, where the source is read as well: 0.98.
bool aligns_source(const hp_plan &p) {
    if (p.dst_copies >= 4 && p.bwd_bytes < 100000000) return false;
    return p.src_copies == 1 ? p.dst_copies == 1 : p.dst_copies <= 2 * p.src_copies;
}

// Against a tile for a row's rest, or for the whole rows that fit, by the share of a
// tile that those fill; the same buffers in turn, two and four samples a position,
// rows of 384 to 12416 bytes, 1 to 16 copies, 40 MB to 2 GB, the direction's gain:
//   forward      share under 0.87: 1.0-1.3 to 450 MB, above 1.0-1.8 (3.5 TB/s at 0.53: to four
//                copies in rows of 2176 bytes, 1.2 GB 327 -> 213 us); more: 0.95-1.0 to 400 MB, 1.0-1.1
//   backward     rows of 1 KiB and more 0.98-1.4; shorter ones 0.96-1.05; share over 0.82, 150 MB 0.96-1.0
//   accumulating 0.98-1.4
// Rows that are not whole lines, in as many lines as they can touch, against tiles that each row cuts
// for itself at lines, or groups of whole rows (0.4 to 21 KB a row, 1 to 16 copies, 30 MB to 1.5 GB), where
// they pay (padding_pays):
//   forward      1.0-1.75 (rows of 4610 bytes to two copies, 0.7 GB 1.61; 2320 bytes to four, 1.5 GB 1.46)
//   backward     0.97-1.7 (1390 bytes from eight copies, 0.5 GB 1.45)
//   accumulating 0.97-1.45
// Rows of a tile and more that fill tiles as well without: 0.8-1.05; groups of rows backward that fill a
// tile to 12 % more: 0.92-1.02, forward to 15 % more still 1.0-1.2, to 15 to 25 % more 0.93-1.02 (rows of 500 bytes, 60 MB to
// 2.5 GB) but in 8 KiB tiles 1.0-1.1.
// The lines that are left out forward lost 3 to 10 %: launches in which partly empty
// tiles happen to leave as much on its way as suits them (two copies, one row in an 8 KiB tile: rows of 4224 to 5120 bytes
// 0.94-0.99 from 150 MB on, 5376 to 7040 0.98-1.0); backward from one copy, rows that
// are not whole chunks and fill three quarters of 2 KiB tiles, 0.91-1.07.
// What is left of such scatter: forward to two to seven copies in rows of 3200, 3456 and 10496 bytes, 0.2 to 1.2 GB, 0.90-0.99,
// and launches of 5 to 25 MB in either direction 0.80-1.2, 1.00 in the middle.
bool cuts_launch(const hp_plan &p, int direction, int variant) {
    if (!p.cut_tiles[variant]) return false;
    if (p.cut_tiles[variant] > p.n_tiles(variant) && p.cut_tiles[variant] >= 1u << 22) return false;   // keep_grid counted the others
    const int64_t row = p.row_bytes, tile = tile_bytes_of(variant), c = p.dst_copies;
    const double share = row_share(row, tile);
    const double bytes = direction == 1 ? (double)p.bwd_bytes : direction == 2 ? (double)p.bwd_accum_bytes
                                                                              : (1.0 + (double)c) * (double)p.n_rows * (double)row;
    if (row % 128) {
        if (!padding_pays(p, variant, direction) || (row < 2048 && bytes < 1e6)) return false;      // (a few tiles: no matter)
        if (direction == 1) return c != 1 || tile != 2048 || share < 0.75 || row % 16 == 0;
        return direction == 2 || c != 8 || tile != 2048 || bytes < 1000e6;
    }
    if (direction == 1) return row >= 1024 && (bytes < 400e6 ? share < 0.82 : share < 0.87 || like_dense(p));
    if (share >= 0.87 && bytes < 400e6) return false;
    if (direction == 2) return true;
    if (c == 2 && tile == 8192 && row < tile && 2 * row > tile && bytes >= 100e6) return false;     // one row a tile, which is as much as suits it
    if ((c == 3 || c == 4) && row >= 1024 && row < 2048 && bytes < 450e6) return false;
    if ((c == 6 || c == 7) && share >= 0.7 && row < 3072 && bytes < 450e6) return false;
    return !eight_short(p, bytes);
}

int build_host_plan(const hp_layout_t *srcs, int32_t n_edges, const hp_layout_t *dst,
                    const hp_token_map_t *maps, int32_t n_maps, hp_plan *p) {
    if (!srcs || !maps || n_maps < 1 || n_edges < 1) return HP_EINVAL;
    int64_t n_bufs = 0;
    for (int32_t e = 0; e < n_edges; ++e) {
        for (int32_t i = 0; i < n_maps; ++i) {
            const hp_token_map_t &m = maps[(size_t)e * n_maps + i];
            int rc = validate(&srcs[e], dst, &m);
            if (rc != HP_OK) return rc;
            // microbatches and edges share the buffer shapes
            if (m.batch != maps[0].batch || m.seq != maps[0].seq || m.hidden != maps[0].hidden ||
                m.dtype != maps[0].dtype)
                return HP_ELAYOUT;
        }
        n_bufs += (int64_t)srcs[e].tp * srcs[e].dp * n_maps;
    }
    n_bufs += (int64_t)dst->tp * dst->cp * dst->dp * n_maps;
    if (n_bufs > HP_MAX_BUFFERS) return HP_ELAYOUT;
    if (n_edges > 1) {
        int rc = check_cross_edge_overlap(maps, n_edges, n_maps);
        if (rc != HP_OK) return rc;
    }
    const hp_token_map_t *m0 = &maps[0];

    p->src = srcs[0];
    p->dst = *dst;
    p->batch = m0->batch; p->seq = m0->seq; p->hidden = m0->hidden; p->dtype = m0->dtype;
    p->n_maps = n_maps;
    p->n_edges = n_edges;
    p->elem_bytes = m0->dtype == HP_F32 ? 4 : 2;
    p->row_bytes = (int64_t)m0->hidden * p->elem_bytes;
    if (p->row_bytes > (int64_t)1 << 24) return HP_ELAYOUT;       // a tile holds whole rows in 32 bits
    const int32_t dst_per_map = dst->tp * dst->cp * dst->dp;
    p->n_dst_bufs = dst_per_map * n_maps;
    p->src_copies = srcs[0].tp;
    p->dst_copies = dst->tp_mode == HP_TP_SEQ_SHARD ? 1 : dst->tp;

    const DstWalker walk(*dst, m0->seq);
    const int64_t b_loc = m0->batch / dst->dp;                     // samples per destination dp rank
    p->dst_rows_per_buf = b_loc * walk.piece;
    const bool sbh = dst->row_order == HP_ROW_SBH;
    const int64_t stride = (sbh && b_loc > 1) ? b_loc : 1;
    p->dst_stride = stride;

    p->n_rows = 0;
    p->bwd_bytes = p->bwd_accum_bytes = 0;
    p->segments.clear();
    p->seg_copies.clear();
    p->src_rows.clear();
    p->src_leader.clear();
    int32_t edge_base = 0;
    for (int32_t e = 0; e < n_edges; ++e) {
        const hp_layout_t *src = &srcs[e];
        const int32_t src_per_map = src->tp * src->dp;
        p->src_rows.resize((size_t)edge_base + (size_t)src_per_map * n_maps, 0);
        p->src_leader.resize(p->src_rows.size(), 0);
        int64_t edge_rows = 0;
        for (int32_t mi = 0; mi < n_maps; ++mi) {
            const hp_token_map_t *m = &maps[(size_t)e * n_maps + mi];
            const int32_t src_base = edge_base + mi * src_per_map, dst_base = mi * dst_per_map;
            // source side: each dp rank's buffer fills up in global image order
            std::vector<int64_t> fill(src->dp, 0);
            const int64_t K = m->n_images;
            int32_t d = 0;
            for (int64_t k = 0; k < K; ++k) {
                if (m->img_src_dp) {
                    d = m->img_src_dp[k];
                } else {
                    while (k >= ((int64_t)(d + 1) * K) / src->dp) ++d;    // next balanced interval
                }
                const int32_t b = m->img_sample[k];
                const int32_t dpd = (int32_t)(b / b_loc);
                const int64_t bl = b - (int64_t)dpd * b_loc;
                int64_t s = m->img_start[k], left = m->img_len[k];
                while (left > 0) {
                    const DstPos pos = walk.at(dpd, s);
                    const int64_t n = std::min(left, pos.run);
                    hp_segment_t seg;
                    seg.src_buf = src_base + d * src->tp;
                    seg.dst_buf0 = dst_base + pos.buf0;
                    seg.src_row0 = fill[d];
                    seg.dst_row0 = sbh ? pos.s_loc * b_loc + bl : bl * walk.piece + pos.s_loc;
                    seg.n_rows = n;
                    seg.dst_row_stride = stride;
                    bool merged = false;
                    if (!p->segments.empty()) {
                        hp_segment_t &q = p->segments.back();
                        if (q.src_buf == seg.src_buf && q.dst_buf0 == seg.dst_buf0 &&
                            q.dst_row_stride == seg.dst_row_stride &&
                            q.src_row0 + q.n_rows == seg.src_row0 &&
                            q.dst_row0 + q.n_rows * q.dst_row_stride == seg.dst_row0 &&
                            q.n_rows + n <= (int64_t)kMaxSegRows) {   // the device descriptor counts rows in 32 bits
                            q.n_rows += n;
                            merged = true;
                        }
                    }
                    if (!merged) {
                        p->segments.push_back(seg);
                        p->seg_copies.push_back(src->tp);
                    }
                    fill[d] += n;
                    edge_rows += n;
                    s += n;
                    left -= n;
                }
            }
            for (int32_t dd = 0; dd < src->dp; ++dd)
                for (int32_t t = 0; t < src->tp; ++t) {
                    p->src_rows[src_base + t + src->tp * dd] = fill[dd];
                    p->src_leader[src_base + t + src->tp * dd] = t == 0;
                }
        }
        p->n_rows += edge_rows;
        const int64_t edge_bytes = edge_rows * p->row_bytes;
        p->bwd_bytes += ((int64_t)p->dst_copies + src->tp) * edge_bytes;
        p->bwd_accum_bytes += (int64_t)p->dst_copies * edge_bytes + (int64_t)src->tp * 2 * edge_rows * p->hidden * 4;
        edge_base += src_per_map * n_maps;
    }
    p->n_src_bufs = edge_base;

    // the launches' shapes ask what can be cut
    const int rc = make_tables(p);
    if (rc == HP_OK) default_launches(p);
    return rc;
}

}  // namespace hp
