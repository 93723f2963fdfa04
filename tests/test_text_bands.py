"""hp_text_grads in [S,B,H] order: the bands of whole positions that it takes for up to 32 samples a buffer."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_27678_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bands_cover_every_row_once(tmp_path):
    exe, csrc = tmp_path / "walk_bands", os.path.join(ROOT, "paper_2605_27678_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-Wall",
                        "-Wno-unknown-pragmas", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                        os.path.join(ROOT, "tests", "walk_bands.cpp"), os.path.join(csrc, "hp_plan.cpp"), "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe), "7", "60"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip() == "plans 60", r.stdout + r.stderr


# samples: a power of two, none, as many as a band has bits, one more (a run for each stretch of each sample); rows:
# whole tiles, pieces with a rest, a little under and over a tile, groups of short ones, not of whole chunks, one element
@pytest.mark.gpu
@pytest.mark.parametrize("samples,hidden,f32", [(4, 4096, False), (3, 2304, False), (2, 2049, False), (4, 1023, True), (3, 2040, False),
                                                (4, 200, False), (5, 67, False), (3, 1, False), (32, 96, True), (33, 96, False)])
def test_text_gradients_in_bands(samples, hidden, f32):
    import torch
    import paper_2605_27678_amd as hp
    rng = np.random.default_rng(samples * hidden)
    seq, tp, samp, start, length = 24, 2, [], [], []
    for b in range(samples):
        at = int(rng.integers(0, 5))
        while at < seq:
            samp, start, length = samp + [b], start + [at], length + [int(min(seq - at, rng.integers(1, 8)))]
            at += length[-1] + int(rng.integers(0, 6))
    tm = wl.TokenMap(samples, seq, hidden, *(np.array(a, np.int32) for a in (samp, start, length)), None, int(f32))
    plan = hp.hp_plan_create(wl.Grid(), wl.Grid(tp=tp, row_order=wl.ROW_SBH), tm)
    g = [torch.randn(samples * seq, hidden, device="cuda").to(torch.float32 if f32 else torch.bfloat16) for _ in range(tp)]
    out, keep = [torch.full_like(t, 7.0) for t in g], [t.clone() for t in g]
    hp.hp_text_grads(plan, g, out)
    image = torch.zeros(seq, samples, dtype=torch.bool)
    for b, s, n in zip(samp, start, length):
        image[s:s + n, b] = True
    image = image.reshape(-1, 1).cuda()
    for t, o, k in zip(g, out, keep):
        assert torch.equal(o, torch.where(image, torch.zeros_like(t), t)) and torch.equal(t, k)
    plan.close()
