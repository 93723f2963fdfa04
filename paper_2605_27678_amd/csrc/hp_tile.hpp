// Internal: what a kernel launch knows about the plan, and how a workgroup finds
// its tile.  Shared by the gfx950 kernels and by a host-side test that walks
// every tile of every launch shape on the CPU (same code, so the index
// arithmetic the GPU runs is checked for bounds without a GPU).
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

#include "hp_plan.hpp"

#if defined(__HIPCC__)
#define HP_HD __host__ __device__ __forceinline__
#else
#define HP_HD inline
#endif

namespace hp {

// Everything else a kernel needs, also by value.
struct KParams {
    uint32_t root[kTreeFanout]; // the top node of this launch's tree: read with the arguments, no load of its own
    const Seg *segs;            // segment descriptors
    const uint32_t *tree;       // search trees (64-byte aligned nodes of 16 keys)
    uint32_t seg_at, tree_at;   // if not 0: the tables travel with the arguments, this many bytes from their start
    uint32_t n_levels;          // levels of this launch's tree
    uint32_t tile_bytes;
    uint32_t row_bytes;
    uint32_t block;             // work-items of a workgroup
    uint32_t dst_base;          // index of the first destination pointer in BufTable
    uint32_t dst_copies;        // replicas of each row on the destination side
    uint32_t parts_per_row;     // row-strided segments, rows of at least a tile: ceil(row_bytes / tile_bytes); else 0
    uint32_t part_magic, part_shift;      // t / parts_per_row = t * part_magic >> (31 + part_shift)
    uint32_t rows_per_tile;     // row-strided segments, rows shorter than a tile: tile_bytes / row_bytes; 0 = cut by bytes or lines, with
                                // the magic number of parts_per_row for a row's lines
    uint32_t row_chunks;        // row-strided tiles of whole rows: lane chunks of one row (see set_row_chunks)
    uint32_t row_magic, row_one;
    uint32_t pace;              // rounds of pace() before a tile's loads (kernels that have it)
    uint32_t level_off[kMaxTreeLevels];   // start of each level, in keys; level 0 = leaves
    uint32_t band_samples, band_magic, band_shift;     // text gradients in bands (band_runs): samples of a position, and their division as above
};

// Device pointers of every buffer of a call, passed by value in the kernel
// argument segment: sources first, destinations from index n_src on.  Lookups
// use wave-uniform indices and become scalar loads.
struct BufTable {
    void *p[HP_MAX_BUFFERS];
};

// The arguments of a transform kernel.  The tables of a plan that leaves the
// room travel behind its buffer pointers (inline_tables), so that an ordinary plan
// of up to about a hundred segments needs no device memory, no upload and, in the
// kernel, no load from memory that the launch itself has not just written.
struct Args {
    KParams k;
    BufTable b;
};
static_assert(sizeof(Args) <= 4096, "kernel arguments");

// One workgroup's share of the launch.
struct TileView {
    uint64_t src_off, dst_off;  // bytes from the buffer bases
    uint32_t nbytes;
    uint32_t pitch_rows;        // 1 = dense destination
    uint32_t row;               // row-strided segments and bands: the tile's (first) row
    uint32_t col;               // cut by bytes or lines: where the tile begins in that row
    uint32_t src_buf, dst_buf0;
    uint32_t src_copies;        // identical TP copies of the source rank
    uint32_t first;             // dense: 1 = the tile starts its run (the segment, or one row of a row-strided one)
    uint64_t left;              // dense: bytes from the tile's start to the end of its run
};

// Tables are read through the scalar cache wherever they lie.
#if defined(__HIP_DEVICE_COMPILE__)
#define HP_TABLE __attribute__((address_space(4)))
#else
#define HP_TABLE
#endif

// One node of the search tree: 16 ascending keys (padding = UINT32_MAX), fetched
// with one 64-byte scalar load; the first is <= tile.  Returns the index of the
// last key that is <= tile, and that key.  Bisected in pairs of keys: four
// compares and eight selects.  What a wave does before its first load is time in
// which it has nothing in flight, at the start of a launch and at every replacement
// of a workgroup.  Against comparing all 16 keys (a hundred instructions), the same
// buffers in turn: to four copies, 100 MB 16.24 -> 16.18 us, 2.06 GB 334 -> 327; from two
// copies, 100 MB 17.2 -> 17.0, 900 MB in 561 segments (three levels) 161 -> 138.  Not
// all gain: the long search spaced out a compute unit's waves, and large launches of
// small tiles with one or two levels lose 1-2 % without it - backward from two and three
// copies 0.98-0.99, where hp::pace_rounds does the same on purpose, forward to two copies
// of 2.5 GB and more 0.99.
template <typename Node>
HP_HD void search_node(Node node, uint32_t tile, uint32_t &index, uint32_t &key) {
    uint64_t q[kTreeFanout / 2];
#pragma unroll
    for (int j = 0; j < 8; ++j) q[j] = (uint64_t)node[2 * j + 1] << 32 | node[2 * j];
    const bool b3 = tile >= (uint32_t)q[4];
    index = b3 ? 8u : 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = b3 ? q[4 + j] : q[j];
    const bool b2 = tile >= (uint32_t)q[2];
    index = b2 ? index + 4u : index;
#pragma unroll
    for (int j = 0; j < 2; ++j) q[j] = b2 ? q[2 + j] : q[j];
    const bool b1 = tile >= (uint32_t)q[1];
    q[0] = b1 ? q[1] : q[0];
    index = b1 ? index + 2u : index;
    const bool b0 = tile >= (uint32_t)(q[0] >> 32);
    key = b0 ? (uint32_t)(q[0] >> 32) : (uint32_t)q[0];
    uint32_t next = index + 1u;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+s"(next));       // a select; the sum with a truth value goes through the vector unit
#endif
    index = b0 ? next : index;
}

// A whole descriptor with one scalar load (left to itself the compiler reads it in
// three, each after a wait for the one before).
HP_HD Seg load_seg(const HP_TABLE Seg *p) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
    u32x8 w = *(const HP_TABLE u32x8 *)p;
    asm("" : "+s"(w));
    return __builtin_bit_cast(Seg, w);
#else
    return *p;
#endif
}

// left < tile ? left : tile, without a 64-bit comparison (the scalar unit has none).
HP_HD uint32_t clip(uint64_t left, uint32_t tile) {
    const uint32_t lo = (uint32_t)left;
    uint32_t hi = (uint32_t)(left >> 32);
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+s"(hi));
#endif
    return hi ? tile : lo < tile ? lo : tile;
}

// What the segments of a launch are; they all have the same pitch, and a kernel's
// variants leave out the other kind.
enum SegKinds {
    kWholeTiles,    // dense, or row-strided with rows of at least a tile
    kRowGroups,     // row-strided with rows shorter than a tile
    kCutRows,       // row-strided, cut by bytes
    kPaddedRows,    // row-strided, cut by lines of the destination
};
constexpr uint32_t kLineBytes = 128;
inline SegKinds seg_kinds(const KParams &k, uint64_t pitch_rows) {
    if (k.rows_per_tile == 0) return k.row_bytes % kLineBytes ? kPaddedRows : kCutRows;
    return pitch_rows != 1 && k.parts_per_row == 0 ? kRowGroups : kWholeTiles;
}

// x / n for x < 2^31, n's magic number and shift made by set_division.
HP_HD uint32_t divide(uint32_t x, uint32_t magic, uint32_t shift) { return (uint32_t)((uint64_t)x * magic >> 31 >> shift); }

// Scalar code: every value here is uniform over the workgroup.  One dependent
// scalar load per tree level below the root, then the descriptor, then the buffer
// pointers.  segs and tree point at k's tables (k.segs and k.tree, or behind the
// arguments).
// BANDS: dense runs that are cut row by row, as row-strided ones are.
template <SegKinds KINDS, bool BANDS = false>
HP_HD TileView locate_tile(const KParams &k, const HP_TABLE Seg *segs, const HP_TABLE uint32_t *tree, uint32_t tile) {
    uint32_t lo, first, index;
    search_node(k.root, tile, lo, first);
#pragma unroll
    for (int l = kMaxTreeLevels - 2; l >= 0; --l) {
        if (__builtin_expect((uint32_t)l + 1 < k.n_levels, l == 0)) {
            search_node(tree + k.level_off[l] + (size_t)lo * kTreeFanout, tile, index, first);
            lo = lo * kTreeFanout + index;
        }
    }
    const Seg s = load_seg(segs + lo);
    const uint32_t t = tile - first;
    TileView v;
    v.pitch_rows = s.pitch_rows;
    v.src_buf = s.src_buf;
    v.dst_buf0 = s.dst_buf0;
    v.src_copies = s.src_copies;
    v.first = t == 0;
    if (KINDS == kWholeTiles && !BANDS && s.pitch_rows == 1) {
        const uint64_t off = (uint64_t)t * k.tile_bytes;
        const uint64_t left = (uint64_t)s.n_rows * k.row_bytes - off;
        v.src_off = s.src_off + off;
        v.dst_off = s.dst_off + off;
        v.nbytes = clip(left, k.tile_bytes);
        v.left = left;
    } else if (KINDS == kWholeTiles) {
        // a piece of one row: dense on both sides, handled like a dense tile
        const uint32_t row = divide(t, k.part_magic, k.part_shift);
        const uint32_t off = (t - row * k.parts_per_row) * k.tile_bytes;
        const uint32_t left = k.row_bytes - off;
        v.pitch_rows = 1;
        v.src_off = s.src_off + (uint64_t)row * k.row_bytes + off;
        v.dst_off = s.dst_off + (uint64_t)row * s.pitch_rows * k.row_bytes + off;
        v.nbytes = left < k.tile_bytes ? left : k.tile_bytes;
        v.first = off == 0;
        v.left = left;
        v.row = row;
    } else if (KINDS == kPaddedRows) {
        const uint32_t row_lines = k.row_bytes / kLineBytes + 2, lines = t * (k.tile_bytes / kLineBytes);
        const uint32_t row0 = divide(lines, k.part_magic, k.part_shift);
        v.col = (lines - row0 * row_lines) * kLineBytes;
        v.src_off = s.src_off + (uint64_t)row0 * k.row_bytes;
        v.dst_off = s.dst_off + (uint64_t)row0 * s.pitch_rows * k.row_bytes;
        v.left = ((uint64_t)s.n_rows * row_lines - lines) * kLineBytes;
        v.nbytes = clip(v.left, k.tile_bytes);
        v.row = row0;
    } else if (KINDS == kCutRows) {
        const uint64_t off = (uint64_t)t * k.tile_bytes;
        const uint32_t row0 = divide(t * (k.tile_bytes / kLineBytes), k.part_magic, k.part_shift);
        v.col = (uint32_t)off - row0 * k.row_bytes;
        v.src_off = s.src_off + off;
        v.dst_off = s.dst_off + (uint64_t)row0 * s.pitch_rows * k.row_bytes + v.col;
        v.left = (uint64_t)s.n_rows * k.row_bytes - off;
        v.nbytes = clip(v.left, k.tile_bytes);
        v.row = row0;
    } else {
        const uint64_t row0 = (uint64_t)t * k.rows_per_tile;
        const uint32_t rows = clip(s.n_rows - row0, k.rows_per_tile);
        v.src_off = s.src_off + row0 * k.row_bytes;
        v.dst_off = s.dst_off + row0 * s.pitch_rows * k.row_bytes;
        v.nbytes = rows * k.row_bytes;
        v.left = v.nbytes;
        v.row = (uint32_t)row0;
    }
    return v;
}

#if !defined(__HIP_DEVICE_COMPILE__)
// The lookup that a launch's kernels have, on the host.
inline TileView locate_tile(const KParams &k, uint32_t tile) {
    switch (seg_kinds(k, k.segs->pitch_rows)) {
        case kRowGroups: return locate_tile<kRowGroups>(k, k.segs, k.tree, tile);
        case kCutRows: return locate_tile<kCutRows>(k, k.segs, k.tree, tile);
        case kPaddedRows: return locate_tile<kPaddedRows>(k, k.segs, k.tree, tile);
        default: return locate_tile<kWholeTiles>(k, k.segs, k.tree, tile);
    }
}
#endif

// Moves both ends of a dense tile up to the next 128-byte line of its first
// destination copy (`dst_base` = that buffer's address), except where its run
// begins and ends: the tiles of a run still partition it, but where rows are no
// multiple of a line, two tiles - two workgroups, on two XCDs with an L2 each -
// no longer share one.  A tile of fewer than 128 bytes may become empty.
HP_HD void align_tile(TileView &v, uint64_t dst_base) {
    if (v.pitch_rows != 1) return;
    const uint32_t up = (uint32_t)(0 - (dst_base + v.dst_off)) & (kLineBytes - 1);
    const uint32_t end = v.left < v.nbytes + up ? (uint32_t)v.left : v.nbytes + up;
    const uint32_t begin = v.first ? 0u : up < end ? up : end;
    v.src_off += begin;
    v.dst_off += begin;
    v.nbytes = end - begin;
}

// Row-strided tiles of whole rows: chunk i of the tile is chunk i % row_chunks of
// row i / row_chunks, in chunks of `unit` bytes.  row_magic = ceil(2^32 / row_chunks)
// divides exactly while i * row_chunks < 2^32 (here i < 2^16 and row_chunks <= 2^13:
// such rows are shorter than the largest tile of 64 KiB); for a single chunk, whose
// magic would not fit, row_one passes i through.
inline void set_row_chunks(KParams &k, uint32_t unit) {
    k.row_chunks = (k.row_bytes + unit - 1) / unit;
    if (k.rows_per_tile == 0 && k.row_bytes % kLineBytes) k.row_chunks = (uint32_t)cut_row_lines(k.row_bytes) * (kLineBytes / unit);
    k.row_one = k.row_chunks == 1 ? ~0u : 0u;
    k.row_magic = k.row_one ? 0u : (uint32_t)((((uint64_t)1 << 32) + k.row_chunks - 1) / k.row_chunks);
}

// Where a lane's chunk lies: bytes from the tile's start on the dense (source)
// side and on the destination side, and how many of its bytes the chunk before
// it covers as well (the last chunk of a run whose length is no multiple of
// the chunk is moved back so that it ends with the run).
struct ChunkView {
    uint64_t dst;
    uint32_t src, over;
    uint32_t end;       // padded rows: bytes before those that the next chunk covers too, else not set
};
// The row of chunk i of a row-strided tile of whole rows.
HP_HD uint32_t row_of_chunk(const KParams &k, uint32_t i) {
    return (uint32_t)(((uint64_t)i * k.row_magic) >> 32) + (i & k.row_one);
}
template <uint32_t UNIT, bool DENSE, bool GUARD>
HP_HD ChunkView chunk_at(const KParams &k, const TileView &t, uint32_t i) {
    ChunkView c;
    if (DENSE) {
        const uint32_t at = i * UNIT, last = t.nbytes - UNIT;
        c.src = GUARD && at > last ? last : at;
        c.over = at - c.src;
        c.dst = c.src;
    } else {
        const uint32_t row = row_of_chunk(k, i);
        const uint32_t at = (i - row * k.row_chunks) * UNIT, last = k.row_bytes - UNIT;
        const uint32_t col = at > last ? last : at;
        c.src = row * k.row_bytes + col;
        c.over = at - col;
        c.dst = (uint64_t)row * t.pitch_rows * k.row_bytes + col;
    }
    return c;
}

// Chunk i of a tile that was cut by bytes: on the source side it lies as in a dense
// tile, on the destination's it has the rest of the positions between its row and the tile's
// first before it.  Rows of a tile and more: their end is passed once at most.
template <uint32_t UNIT>
HP_HD ChunkView cut_chunk(const KParams &k, const TileView &t, uint32_t i) {
    ChunkView c;
    c.src = i * UNIT;
    c.over = 0;
    const uint64_t gap = (uint64_t)(t.pitch_rows - 1) * k.row_bytes;
    if (k.row_bytes >= k.tile_bytes) c.dst = c.src + (t.col + c.src >= k.row_bytes ? gap : 0);
    else c.dst = c.src + row_of_chunk(k, i + t.col / UNIT) * gap;
    return c;
}

// Chunk i of a tile that was cut by lines of the destination, `dst_line` = the address
// of the tile's first row there: from the row's start, which the tile's offsets are those
// of.  A row has room for all the lines that it can touch; a chunk of which no byte is its
// row's is not there (false), and those at the row's ends are moved to begin and
// end with it, over bytes of their neighbours.  Rows of kMinPaddedRow bytes and more.  All of a
// wave's lanes but those at the ends then store to whole 64-byte pieces: stores that begin
// between them take half as long again (four copies, 283 MB: 42 -> 67 us).
template <uint32_t UNIT>
HP_HD bool padded_chunk(const KParams &k, const TileView &t, uint32_t dst_line, uint32_t i, ChunkView &c) {
    const uint32_t j = i + t.col / UNIT;
    const uint32_t row = row_of_chunk(k, j);
    const uint32_t skip = (dst_line + row * t.pitch_rows * k.row_bytes) & (kLineBytes - 1);
    const int32_t at = (int32_t)((j - row * k.row_chunks) * UNIT) - (int32_t)skip, last = (int32_t)k.row_bytes - (int32_t)UNIT;
    const uint32_t in_row = (uint32_t)(at < 0 ? 0 : at > last ? last : at);
    c.src = row * k.row_bytes + in_row;
    c.dst = (uint64_t)row * t.pitch_rows * k.row_bytes + in_row;
    c.over = at > last ? (uint32_t)(at - last) : 0u;
    c.end = at < 0 ? UNIT - (uint32_t)-at : UNIT;
    return at > -(int32_t)UNIT && at < (int32_t)k.row_bytes;
}

// How many chunks of UNIT bytes a tile has, and how many of them lie in their
// run as they are (those before the moved one).  0 chunks: the run is shorter
// than a chunk and is walked element by element.
template <uint32_t UNIT, bool DENSE>
HP_HD void count_chunks(const KParams &k, const TileView &t, uint32_t &all, uint32_t &whole) {
    if (DENSE) {
        all = t.nbytes >= UNIT ? (t.nbytes + UNIT - 1) / UNIT : 0u;
        whole = all ? t.nbytes / UNIT : 0u;
    } else {
        all = whole = k.row_bytes >= UNIT ? t.nbytes / k.row_bytes * k.row_chunks : 0u;
    }
}

// The walk one element at a time (ELEM bytes): element i of the tile.
template <uint32_t ELEM>
HP_HD ChunkView element_at(const KParams &k, const TileView &t, uint32_t i) {
    ChunkView c;
    const uint32_t at = i * ELEM;
    c.src = at;
    c.over = 0;
    if (t.pitch_rows == 1) c.dst = at;
    else {
        const uint32_t row = at / k.row_bytes;
        c.dst = (uint64_t)row * t.pitch_rows * k.row_bytes + (at - row * k.row_bytes);
    }
    return c;
}

// Multiplication in place of x / n, exact for x < 2^31 (a grid has no
// more tiles): with 2^shift >= n the magic number, rounded up, is off by
// less than 2^shift in 2^(31 + shift).  The division itself, some 30
// instructions of the vector unit and a read back from it, stood before the first
// load of every piece of a row.
inline void set_division(uint32_t n, uint32_t &magic, uint32_t &shift) {
    magic = shift = 0;
    if (!n) return;
    while ((1u << shift) < n) ++shift;
    magic = (uint32_t)((((uint64_t)1 << (31 + shift)) + n - 1) / n);
}
inline void set_parts(KParams &k) { set_division(k.parts_per_row, k.part_magic, k.part_shift); }

// Text gradients in bands: the sample (0 .. band_samples - 1) of a run's row, less than 2^31.
HP_HD uint32_t band_sample(const KParams &k, uint32_t row) {
    return row - divide(row, k.band_magic, k.band_shift) * k.band_samples;
}

// The kernel parameters of a launch with tiles of 1 KiB << variant; segs and
// tree point at the plan's tables wherever the caller keeps them (device memory
// for a launch, the plan's host vectors for the host-side walk).
// cut: for the launch that cuts row-strided segments by bytes, where the plan has one.
inline KParams kernel_params(const hp_plan &p, int variant, const Seg *segs, const uint32_t *tree, bool cut = false) {
    KParams k;
    const TreeInfo &ti = cut ? p.cut_info[variant] : p.tree_info[variant];
    for (int j = 0; j < kTreeFanout; ++j)
        k.root[j] = ti.n_levels ? p.tree[ti.level_off[ti.n_levels - 1] + j] : UINT32_MAX;
    k.segs = segs;
    k.tree = tree;
    k.seg_at = k.tree_at = 0;
    k.n_levels = ti.n_levels;
    for (int l = 0; l < kMaxTreeLevels; ++l) k.level_off[l] = ti.level_off[l];
    k.tile_bytes = tile_bytes_of(variant);
    k.row_bytes = (uint32_t)p.row_bytes;
    k.rows_per_tile = std::max<uint32_t>(1u, k.tile_bytes / k.row_bytes);
    k.parts_per_row = k.row_bytes >= k.tile_bytes ? (k.row_bytes + k.tile_bytes - 1) / k.tile_bytes : 0u;
    set_parts(k);
    if (cut) {
        k.parts_per_row = k.rows_per_tile = 0;
        set_division((uint32_t)cut_row_lines(p.row_bytes), k.part_magic, k.part_shift);
    }
    set_row_chunks(k, 16u);
    k.block = k.pace = 0;       // set by the launch
    k.band_samples = k.band_magic = k.band_shift = 0;      // by that of text gradients in bands
    k.dst_base = (uint32_t)p.n_src_bufs;
    k.dst_copies = (uint32_t)p.dst_copies;
    return k;
}

// Where the tables begin behind a plan's buffer pointers in a launch's arguments, and whether those of n of its
// segments fit there.
inline size_t inline_seg_at(const hp_plan &p) {
    return (offsetof(Args, b) + (size_t)(p.n_src_bufs + p.n_dst_bufs) * sizeof(void *) + 63) / 64 * 64;
}
inline bool inline_fits(const hp_plan &p, size_t n) {
    const size_t leaves = n > (size_t)kTreeFanout ? (n + kTreeFanout - 1) / kTreeFanout * 64 : 0;
    return inline_seg_at(p) + (n * sizeof(Seg) + 63) / 64 * 64 + leaves <= sizeof(Args);
}

// A launch of hp_forward_static that writes tables into the device's array first takes a kernel for each of these.
constexpr uint32_t kChunkWords = 896;                       // 3584 bytes, under the 4 KiB argument limit

// How many launches hp_forward_static takes for a plan of several, each of which brings a part of the segments; 0: the
// tables are written into the device's array instead, `tree_bytes` of them the search tree.  Several launches are
// taken where they are no more than the kernels that would write the tables and the one that reads them: 120
// segments, 2.8 MB, 19.6 -> 11.0 us; 400 segments, 192 MB 40.4 -> 35.3; 1000 segments, 46 MB 52.8 -> 46.7.  A launch
// has room for about (3584 - 8 buffers) / 36 segments and a kernel writes 98 to 112, so that it depends on both: plans of up to 18
// buffers always take several launches, others write the tables from about 1570 segments on with 19 buffers, 1440
// with 28, 660 with 60, 450 with 100, 320 with 150 and 90 with 300 (and a few hundred more alternate with the
// rounding up of either).  At hundreds of buffers the two are within 1 %.
inline size_t static_launches(const hp_plan &p, size_t tree_bytes) {
    const size_t chunk = kChunkWords * sizeof(uint32_t), n = p.dsegs.size();
    const size_t most = (n * sizeof(Seg) + chunk - 1) / chunk + (tree_bytes + chunk - 1) / chunk + 1;
    for (size_t launches = 1; launches <= std::min(n, most); ++launches)
        if (inline_fits(p, (n + launches - 1) / launches)) return launches;
    return 0;
}

// One launch of the text-gradient kernel: `n` of the runs from `runs` on, whose
// buffers are the `bufs` from `buf0` on; its tables always travel with the
// arguments.
struct RunGroup {
    size_t first, n;
    int32_t buf0, bufs;
};
inline size_t run_bytes(size_t n, int32_t bufs) {
    const size_t ptrs = (offsetof(Args, b) + (size_t)bufs * 2 * sizeof(void *) + 63) / 64 * 64;
    const size_t leaves = n > (size_t)kTreeFanout ? (n + kTreeFanout - 1) / kTreeFanout * 64 : 0;
    return ptrs + (n * sizeof(Seg) + 63) / 64 * 64 + leaves;
}
// As many runs a launch as the arguments hold.
inline std::vector<RunGroup> group_runs(const std::vector<Seg> &runs, int32_t copies) {
    std::vector<RunGroup> groups;
    for (size_t i = 0; i < runs.size(); ++i) {
        const int32_t buf0 = runs[i].dst_buf0;
        if (!groups.empty()) {
            RunGroup &g = groups.back();
            const int32_t bufs = buf0 + copies - g.buf0;
            if (run_bytes(g.n + 1, bufs) <= sizeof(Args)) {
                ++g.n;
                g.bufs = bufs;
                continue;
            }
        }
        groups.push_back(RunGroup{i, 1, buf0, copies});
    }
    return groups;
}

// Whether the runs of text and image rows are bands: in [S,B,H] order, for as many samples as a band has bits.
inline bool text_bands(const hp_plan &p) { return p.dst_stride > 1 && p.dst_stride <= kMaxBandSamples; }

// The runs that hp_text_grads launches for a plan: of text and of image rows, or
// (*whole) whole buffers to copy, whose image rows are then zeroed.  Runs save the
// image rows one reading and one writing, about 1 us for 6 MB, and take a launch
// for every hundred or so, about 4 us each after the first; a copy is two launches.
// Two buffers of 67 MB, half of them image rows: 512 runs 56 us, 800 runs 67, copied
// 53; 1000 images in two buffers of 34 MB: 99 against 30; two of 524 MB: 4096 runs
// 441 us, 5120 row-strided ones 589, copied 476 and 481.
inline std::vector<Seg> text_runs(const hp_plan &p, bool *whole) {
    const double saved = 2.0 * (double)p.n_rows * (double)p.row_bytes * p.dst_copies;
    const double most = 1.75 + saved / 25e6;                             // launches
    // About as many runs as there will be at least (segments in another order than their rows count as apart): where
    // they are too many they are not even made.  Samples share the bands of images that lie where those of the sample
    // before them do, as under one template for all; others, scattered, hardly any.  4 samples of 120 images in two buffers
    // of 39 MB 32.8 -> 25.8 us, 16 of 64 in 67 MB 57 -> 34, 4 of 400 in 262 MB 211 -> 153; where bands save less than
    // 30 MB the copy is as fast or faster (two of 11 MB, rows of 2304 bytes, 12.2 -> 14.2).
    const int64_t samples = p.dst_stride;
    int64_t images = 0;
    bool alike = text_bands(p) && saved >= 30e6;
    size_t before = 0, first = 0;                                        // where the segments of the sample before and of this one begin,
    int64_t earlier = 0, sample = 0;                                     // and which samples these are
    for (size_t i = 0; i < p.segments.size(); ++i) {
        const hp_segment_t &b = p.segments[i], &a = p.segments[i ? i - 1 : 0];
        images += !i || a.dst_buf0 != b.dst_buf0 || a.dst_row0 + a.n_rows * a.dst_row_stride != b.dst_row0;
        if (!alike) continue;
        const int64_t now = b.dst_row0 % samples;
        if (now != sample) before = first, first = i, earlier = sample, sample = now;
        if (sample == 0) continue;
        const hp_segment_t &o = p.segments[before + (i - first)];
        alike = before + (i - first) < first && o.dst_buf0 == b.dst_buf0 && o.n_rows == b.n_rows && b.dst_row0 - o.dst_row0 == sample - earlier;
    }
    const int64_t columns = p.n_dst_bufs / p.dst_copies * p.dst_stride;
    int64_t runs = std::max(columns, std::max(images, 2 * images - columns));
    if (alike) runs = (runs + samples - 1) / samples;
    if (text_bands(p)) runs = std::min(runs, columns / p.dst_stride * (p.dst_rows_per_buf / p.dst_stride));
    *whole = images == 0 || (double)runs * sizeof(Seg) > most * sizeof(Args);
    if (!*whole) {
        std::vector<Seg> r = text_bands(p) ? band_runs(p) : dst_runs(p, false);
        *whole = (double)group_runs(r, p.dst_copies).size() > most;
        if (!*whole) return r;
    }
    return dst_runs(p, true);
}

}  // namespace hp
