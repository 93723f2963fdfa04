"""hp_backward in tiles that end on lines of the source: ragged rows, one copy to one or few copies to several."""
import numpy as np
import pytest

import paper_2605_27678_amd as hp
from paper_2605_27678_amd import workloads as wl

pytestmark = pytest.mark.gpu


# one copy of each; fewer, as many and more destination copies than source copies; dense runs, pieces of row-strided rows,
# runs of less than a line; buffers that begin anywhere
@pytest.mark.parametrize("tp_src,tp,hidden,sbh,f32", [(1, 1, 2305, False, False), (2, 1, 33, False, False), (2, 2, 1004, False, True), (3, 2, 4094, True, False),
                                                      (2, 3, 71, False, False), (1, 1, 4095, True, True), (2, 1, 3, False, False)])
def test_backward_on_lines_of_the_source(tp_src, tp, hidden, sbh, f32):
    import torch
    from oracle import oracle
    rng = np.random.default_rng(hidden)
    src, dst = wl.Grid(tp=tp_src, dp=2), wl.Grid(tp=tp, cp=2, row_order=wl.ROW_SBH if sbh else wl.ROW_BSH)
    tm = wl.token_map_from_lens(rng, 2, 80, hidden, [[1, 40, 17], [30, 1, 29]])
    tm.dtype = wl.DT_F32 if f32 else wl.DT_BF16
    plan, prob = hp.hp_plan_create(src, dst, tm), oracle.Problem(src, dst, tm)

    def device(t, first):
        big = torch.empty(t.numel() + first, dtype=t.dtype, device="cuda")
        return big[first:].view(t.shape).copy_(t)

    def bits(t):
        t = t.cpu().contiguous()
        return t.numpy().copy() if f32 else t.view(torch.int16).numpy().view(np.uint16).copy()

    kind = torch.float32 if f32 else torch.bfloat16
    g = [torch.from_numpy(rng.standard_normal((prob.dst_rows(), hidden), dtype=np.float32)).to(kind) for _ in range(prob.n_dst)]
    y = [torch.zeros((r, hidden), dtype=kind) for r in prob.src_rows()]
    want = [bits(t) for t in y]
    (prob.backward_f32 if f32 else prob.backward_bf16)([bits(t) for t in g], want)
    G = [device(t, 7 * i % 64) for i, t in enumerate(g)]
    for tile in (1024, 2048, 4096):
        plan.set_launch(1, tile_bytes=tile, block_threads=64)
        out = [device(t, 5 * (i + 1) % 64) for i, t in enumerate(y)]
        hp.hp_backward(plan, G, out)
        for i, (t, w) in enumerate(zip(out, want)):
            assert np.array_equal(bits(t).view(np.uint8), w.reshape(t.shape).view(np.uint8)), (i, tile)
    plan.close()


def _device(t, first):
    import torch
    big = torch.empty(t.numel() + first, dtype=t.dtype, device="cuda")
    return big[first:].view(t.shape).copy_(t)


def _bits(t):
    import torch
    t = t.cpu().contiguous()
    return t.numpy().copy() if t.dtype == torch.float32 else t.view(torch.int16).numpy().view(np.uint16).copy()


def _values(shape, f32, seed):
    import torch
    return torch.randn(shape, generator=torch.Generator().manual_seed(seed)).to(torch.float32 if f32 else torch.bfloat16)


# from four destination copies on it takes launches of 100 MB: the kernels for four and eight copies and for any number, with and without a rest of a group of four; dense
# runs and pieces of row-strided rows
@pytest.mark.parametrize("tp_src,tp,hidden,rows,sbh,f32", [(2, 4, 4095, 2100, False, False), (2, 4, 2049, 2100, True, True), (4, 8, 4094, 1100, True, False), (4, 8, 1027, 2200, False, True),
                                                           (3, 5, 2305, 2800, False, False), (3, 6, 4095, 700, False, True), (8, 16, 1001, 2200, False, False)])
def test_large_launches_on_lines_of_the_source(tp_src, tp, hidden, rows, sbh, f32):
    from oracle import oracle
    rng = np.random.default_rng(hidden)
    samples = 2 if sbh else 1
    cuts = np.sort(rng.integers(1, rows // samples, 6))
    lens = np.diff(np.concatenate([[0], cuts, [rows // samples]]))
    src, dst = wl.Grid(tp=tp_src), wl.Grid(tp=tp, row_order=wl.ROW_SBH if sbh else wl.ROW_BSH)
    tm = wl.token_map_from_lens(rng, samples, rows // samples + 40, hidden, [[int(n) for n in lens if n]] * samples)
    tm.dtype = wl.DT_F32 if f32 else wl.DT_BF16
    plan, prob = hp.hp_plan_create(src, dst, tm), oracle.Problem(src, dst, tm)
    assert plan.info.bwd_bytes >= 100e6 and tp <= 2 * tp_src       # where the rule has them
    g = [_values((prob.dst_rows(), hidden), f32, j) for j in range(prob.n_dst)]
    want = [np.zeros((r, hidden), np.float32 if f32 else np.uint16) for r in prob.src_rows()]
    (prob.backward_f32 if f32 else prob.backward_bf16)([_bits(t) for t in g], want)
    G = [_device(t, 7 * i % 64) for i, t in enumerate(g)]
    for shape in ({}, dict(tile_bytes=4096, block_threads=256)):
        plan.set_launch(1, **shape)
        out = [_device(_values((r, hidden), f32, 9), 5 * (i + 1) % 64) for i, r in enumerate(prob.src_rows())]
        hp.hp_backward(plan, G, out)
        for i, (t, w) in enumerate(zip(out, want)):
            assert np.array_equal(_bits(t).view(np.uint8), w.reshape(t.shape).view(np.uint8)), (i, shape)
    plan.close()


# edges of other numbers of source copies than the first, which the rule goes by: more of them, and fewer
@pytest.mark.parametrize("tps,tp,hidden", [((2, 1), 2, 1003), ((1, 3), 1, 2305), ((1, 2, 1), 1, 71), ((3, 1), 5, 4095)])
def test_joined_edges_on_lines_of_the_source(tps, tp, hidden):
    from oracle import oracle
    rng = np.random.default_rng(hidden)
    seq, n, big = 1500 if tp > 3 else 90, len(tps), tp > 3
    dst = wl.Grid(tp=tp, cp=2, cp_split=wl.CP_ZIGZAG)
    srcs = [wl.Grid(tp=t, dp=1 + e % 2) for e, t in enumerate(tps)]
    unit = seq // (4 * n)
    maps = [[wl.TokenMap(2, seq - seq % 4, hidden, np.repeat([0, 1], 4).astype(np.int32), np.tile(unit * (n * np.arange(4) + e), 2).astype(np.int32),
                         rng.integers(unit - 2 if big else 1, unit + 1 if big else unit, 8).astype(np.int32))] for e in range(n)]
    plan = hp.hp_plan_create_joined(srcs, dst, maps)
    assert not big or plan.info.bwd_bytes >= 100e6
    probs = [oracle.Problem(s, dst, m[0]) for s, m in zip(srcs, maps)]
    g = [_values((probs[0].dst_rows(), hidden), False, j) for j in range(probs[0].n_dst)]
    want = []
    for p in probs:
        w = [np.zeros((r, hidden), np.uint16) for r in p.src_rows()]
        p.backward_bf16([_bits(t) for t in g], w)
        want += w
    out = [_device(_values((len(w), hidden), False, 9), 5 * (i + 1) % 64) for i, w in enumerate(want)]
    hp.hp_backward(plan, [_device(t, 7 * i % 64) for i, t in enumerate(g)], out)
    for i, (t, w) in enumerate(zip(out, want)):
        assert np.array_equal(_bits(t), w), i
    plan.close()
