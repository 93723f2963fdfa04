"""Row-strided segments ([S,B,H] order) of launches that cut them by bytes or by lines, across the ends of rows."""
import os
import subprocess

import numpy as np
import pytest

import paper_2605_27678_amd as hp
from paper_2605_27678_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_chunk_lies_where_its_row_does(tmp_path):
    exe, csrc = tmp_path / "walk_cut", os.path.join(ROOT, "paper_2605_27678_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-Wall",
                        "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", "walk_cut.cpp"), os.path.join(csrc, "hp_plan.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe), "11", "60"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip() == "plans 60", r.stdout + r.stderr


@pytest.mark.parametrize("hidden,tile,cut", [(1280, 2048, True), (1280, 4096, True), (1088, 1024, True), (2048, 1024, False), (4096, 8192, False),
                                             (3072, 1024, False), (640, 4096, False)])
def test_tiles_of_a_launch_that_cuts_its_rows_are_whole(hidden, tile, cut):
    tm = wl.TokenMap(2, 64, hidden, [0, 1], [3, 5], [41, 52])
    p = hp.hp_plan_create_host(wl.Grid(), wl.Grid(row_order=wl.ROW_SBH), tm)
    p.set_launch(0, tile_bytes=tile)
    whole = sum(-(-s.n_rows * 2 * hidden // tile) for s in p.segments())
    pieces = sum(s.n_rows * -(-2 * hidden // tile) if 2 * hidden >= tile else -(-s.n_rows // (tile // (2 * hidden))) for s in p.segments())
    assert p.info.n_tiles == (whole if cut else pieces)
    p.close()


def test_grids_of_the_largest_padded_launches_stay_below_2_to_the_32_work_items():
    # the shape that such a plan starts from, in tiles of 4 KiB; where lines would be too many: test_cut_rules.py
    hidden, rows = 200, (62 << 30) // 400
    tm = wl.TokenMap(2, rows // 2, hidden, [0, 1], [0, 0], [rows // 2] * 2)
    p = hp.hp_plan_create_host(wl.Grid(), wl.Grid(row_order=wl.ROW_SBH), tm)
    assert p.info.n_tiles * p.get_launch(0)["block_threads"] < 2 ** 32
    p.close()


# rows of 384 bytes to 6 KiB, each in tiles that they fill badly, whole lines and not; buffers that begin anywhere; copies with a kernel of their own and without, two
# source copies; the walk through a launch's own arguments and, with many images, through device memory
@pytest.mark.gpu
@pytest.mark.parametrize("tp,hidden,f32,images", [(1, 1280, False, 3), (2, 192, False, 60), (3, 1088, False, 3), (4, 2304, False, 60), (5, 640, False, 3),
                                                  (8, 192, True, 3), (8, 1088, False, 60), (16, 320, True, 3),
                                                  (1, 1025, False, 60), (2, 1544, False, 3), (3, 2305, False, 3), (4, 1027, True, 60), (6, 1100, False, 3),
                                                  (8, 3001, False, 3), (12, 515, True, 3), (1, 695, False, 300), (3, 301, False, 300), (8, 195, True, 300)])
def test_cut_launches(tp, hidden, f32, images):
    import torch
    from oracle import oracle
    rng = np.random.default_rng(100 * tp + hidden)
    src, dst = wl.Grid(tp=2, dp=2), wl.Grid(tp=tp, cp=2, row_order=wl.ROW_SBH)
    lens = [[1, 40, 17], [30, 29], [77]] if images == 3 else [list(rng.integers(1, 4, images)) for _ in range(3)]
    tm = wl.token_map_from_lens(rng, 3, 80 if images == 3 else 400 if images == 60 else 1500, hidden, lens)     # 300: more than 1 MB
    tm.dtype = wl.DT_F32 if f32 else wl.DT_BF16
    plan, host, prob = hp.hp_plan_create(src, dst, tm), hp.hp_plan_create_host(src, dst, tm), oracle.Problem(src, dst, tm)
    rows, drows = prob.src_rows(), prob.dst_rows()
    kind = torch.float32 if f32 else torch.bfloat16

    def values(r, dt=kind):
        return torch.from_numpy(rng.standard_normal((r, hidden), dtype=np.float32)).to(dt)

    def bits(t):
        t = t.cpu().contiguous()
        return t.numpy().copy() if t.dtype == torch.float32 else t.view(torch.int16).numpy().view(np.uint16).copy()

    x, d, g = [values(r) for r in rows], [values(drows) for _ in range(prob.n_dst)], [values(drows) for _ in range(prob.n_dst)]
    y, a = [values(r) for r in rows], [values(r, torch.float32) for r in rows]
    want_d, want_z, want_y, want_a = [bits(t) for t in d], [bits(t) for t in d], [bits(t) for t in y], [bits(t) for t in a]
    prob.forward([bits(t) for t in x], want_d)
    (prob.backward_f32 if f32 else prob.backward_bf16)([bits(t) for t in g], want_y)
    prob.backward_accumulate([bits(t) for t in g], want_a)
    for j, z in enumerate(want_z):
        z.reshape(drows, hidden)[prob.forward_map(j)[0] >= 0] = 0
    def device(t, first):
        big = torch.empty(t.numel() + first, dtype=t.dtype, device="cuda")
        return big[first:].view(t.shape).copy_(t)

    x, d, g, y, a = ([device(t, 5 * (i + 2) % 64) for i, t in enumerate(ts)] for ts in (x, d, g, y, a))
    for shape in ({}, dict(tile_bytes=1024, block_threads=64), dict(tile_bytes=2048, block_threads=64), dict(tile_bytes=4096, block_threads=256),
                  dict(tile_bytes=8192, block_threads=128)):
        for direction in range(3):
            plan.set_launch(direction, **shape)
        host.set_launch(0, **shape)
        out = [[device(t, 3 * i % 64) for i, t in enumerate(ts)] for ts in (d, d, d, y, a)]
        hp.hp_forward(plan, x, out[0])
        hp.hp_forward_static(host, x, out[1])
        hp.hp_zero_image_rows(plan, out[2])
        hp.hp_backward(plan, g, out[3])
        hp.hp_backward_accumulate(plan, g, out[4])
        for what, got, want in zip(("forward", "static", "zero", "backward", "accumulate"), out, (want_d, want_d, want_z, want_y, want_a)):
            for i, (t, w) in enumerate(zip(got, want)):
                assert np.array_equal(bits(t).view(np.uint8), w.reshape(t.shape).view(np.uint8)), (what, i, shape)
    plan.close()
    host.close()
