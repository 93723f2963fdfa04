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
