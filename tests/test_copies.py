"""Every replica count through every kind of tile: the kernels of a fixed count (1, 2, 3, 4, 8), and the one that takes
groups of four and a last group of one to three.  Bit for bit against the oracle; whole and partial tiles, two source copies."""
import numpy as np
import pytest
import torch

import paper_2605_27678_amd as hp
from oracle import oracle
from paper_2605_27678_amd import workloads as wl

pytestmark = pytest.mark.gpu


# hidden 64: rows of lines; 520 in [S,B,H] order: pieces of rows (1040 and 2080 bytes); 33: ragged; 24 in [S,B,H] order: groups of rows
@pytest.mark.parametrize("hidden,sbh", [(64, False), (520, True), (33, False), (24, True)])
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("tp", range(1, 17))
def test_replica_counts_of_every_kind_of_tile(tp, f32, hidden, sbh):
    rng = np.random.default_rng(100 * tp + hidden)
    src, dst = wl.Grid(tp=2, dp=2), wl.Grid(tp=tp, cp=2, row_order=wl.ROW_SBH if sbh else wl.ROW_BSH)
    tm = wl.token_map_from_lens(rng, 2, 80, hidden, [[1, 40, 17], [30, 29]])
    tm.dtype = wl.DT_F32 if f32 else wl.DT_BF16
    plan, prob = hp.hp_plan_create(src, dst, tm), oracle.Problem(src, dst, tm)
    rows, drows = prob.src_rows(), prob.dst_rows()
    kind = torch.float32 if f32 else torch.bfloat16

    def values(r, dt=kind):
        return torch.from_numpy(rng.standard_normal((r, hidden), dtype=np.float32)).to(dt)

    def bits(t):
        t = t.cpu().contiguous()
        return t.numpy().copy() if t.dtype == torch.float32 else t.view(torch.int16).numpy().view(np.uint16).copy()

    x, d, g = [values(r) for r in rows], [values(drows) for _ in range(prob.n_dst)], [values(drows) for _ in range(prob.n_dst)]
    y, a = [values(r) for r in rows], [values(r, torch.float32) for r in rows]
    want_d, want_y, want_a = [bits(t) for t in d], [bits(t) for t in y], [bits(t) for t in a]
    prob.forward([bits(t) for t in x], want_d)
    (prob.backward_f32 if f32 else prob.backward_bf16)([bits(t) for t in g], want_y)
    prob.backward_accumulate([bits(t) for t in g], want_a)
    x, d, g, y, a = ([t.cuda() for t in ts] for ts in (x, d, g, y, a))
    for shape in ({}, dict(tile_bytes=2048, block_threads=64), dict(tile_bytes=1024, block_threads=256)):
        for direction in range(3):
            plan.set_launch(direction, **shape)
        out = [[t.clone() for t in ts] for ts in (d, y, a)]
        hp.hp_forward(plan, x, out[0])
        hp.hp_backward(plan, g, out[1])
        hp.hp_backward_accumulate(plan, g, out[2])
        for what, got, want in zip(("forward", "backward", "accumulate"), out, (want_d, want_y, want_a)):
            for i, (t, w) in enumerate(zip(got, want)):
                assert np.array_equal(bits(t).view(np.uint8), w.reshape(t.shape).view(np.uint8)), (what, i, shape)
    plan.close()


# Launches that are paced (hp::pace_rounds): large ones in tiles of 1 KiB, by the levels of the search tree.
@pytest.mark.parametrize("tp,mbytes,images", [(2, 410, 40), (3, 460, 9), (3, 460, 40), (3, 460, 300), (4, 410, 9), (4, 410, 300), (6, 820, 40),
                                              (16, 220, 9), (16, 220, 40)])
def test_paced_launches(tp, mbytes, images):
    hidden = 2048
    n = mbytes * 1000000 // ((tp + 1) * hidden * 2) // images + 1
    start = [i * (n + 3) for i in range(images)]
    tm = wl.TokenMap(1, images * (n + 3), hidden, [0] * images, start, [n] * images)
    src, dst = wl.Grid(), wl.Grid(tp=tp)
    plan, prob = hp.hp_plan_create(src, dst, tm), oracle.Problem(src, dst, tm)
    gen = torch.Generator(device="cuda").manual_seed(tp * images)

    def values(r):
        return torch.randn((r, hidden), generator=gen, device="cuda", dtype=torch.bfloat16)

    def bits(t):
        return t.cpu().contiguous().view(torch.int16).numpy().view(np.uint16)

    x, g = [values(r) for r in prob.src_rows()], [values(prob.dst_rows()) for _ in range(prob.n_dst)]
    d, y = [torch.zeros_like(t) for t in g], [torch.empty_like(t) for t in x]
    assert (plan.info.n_segments, plan.get_launch(0 if tp == 16 else 1)["tile_bytes"]) == (images, 1024)
    hp.hp_forward(plan, x, d)
    hp.hp_backward(plan, g, y)
    want_d, want_y = [np.zeros(tuple(t.shape), np.uint16) for t in d], [np.zeros(tuple(t.shape), np.uint16) for t in y]
    prob.forward([bits(t) for t in x], want_d)
    prob.backward_bf16([bits(t) for t in g], want_y)
    for got, want in list(zip(d, want_d)) + list(zip(y, want_y)):
        assert np.array_equal(bits(got), want)
    plan.close()
