"""Rows and buffers that no vector width divides: the ragged and the row-strided kernels at the sizes where a chunk,
a line or a tile ends inside a row.  Bit for bit against the oracle, with guards around every buffer."""
import numpy as np
import pytest
import torch

import paper_2605_27678_amd as hp
from oracle import oracle
from paper_2605_27678_amd import workloads as wl

pytestmark = pytest.mark.gpu
GUARD = 192                  # elements before and after every buffer


class Padded:
    """A [rows, hidden] buffer inside a larger one, `off` elements after a 256-byte boundary."""

    def __init__(self, values, off):
        flat = values.reshape(-1)
        self.n, self.at = flat.size, GUARD + off
        self.whole = np.full(self.at + self.n + GUARD, 0x5A, flat.dtype)
        self.whole[self.at:self.at + self.n] = flat
        signed = self.whole.view({2: np.int16, 4: np.int32}[flat.itemsize])
        self.dev = torch.from_numpy(signed).cuda()
        kind = torch.bfloat16 if flat.dtype == np.uint16 else torch.float32
        self.t = self.dev[self.at:self.at + self.n].view(kind).view(values.shape)

    def check(self, want, what):
        got = self.dev.cpu().numpy().view(self.whole.dtype)
        assert np.array_equal(got[:self.at], self.whole[:self.at]), (what, "bytes before the buffer")
        assert np.array_equal(got[self.at + self.n:], self.whole[self.at + self.n:]), (what, "bytes after the buffer")
        assert np.array_equal(got[self.at:self.at + self.n].view(np.uint8), want.reshape(-1).view(np.uint8)), what


# hidden: below a chunk (1, 3, 7), a chunk and its neighbours, around a line, around tiles of 1 and 2 KiB
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("hidden,tp,sbh,off", [(1, 2, True, 0), (3, 3, False, 1), (7, 4, True, 3), (8, 8, True, 1),
                                               (9, 1, False, 5), (63, 4, False, 0), (65, 2, True, 1), (511, 5, True, 0),
                                               (513, 4, False, 7), (1001, 16, False, 1), (1025, 2, True, 2),
                                               (64, 4, False, 1)])
def test_ragged_rows_and_buffers(hidden, tp, sbh, off, f32):
    rng = np.random.default_rng(hidden * 31 + tp)
    src = wl.Grid(tp=2, dp=3)
    dst = wl.Grid(tp=tp, cp=2, dp=1, cp_split=wl.CP_ZIGZAG, row_order=wl.ROW_SBH if sbh else wl.ROW_BSH)
    tm = wl.token_map_from_lens(rng, 2, 48, hidden, [[1, 9, 17, 2], [30, 5]])
    tm.dtype = wl.DT_F32 if f32 else wl.DT_BF16
    plan, prob = hp.hp_plan_create(src, dst, tm), oracle.Problem(src, dst, tm)
    rows, drows = prob.src_rows(), prob.dst_rows()

    def values(r):
        x = torch.from_numpy(rng.standard_normal((r, hidden), dtype=np.float32))
        return x.numpy() if f32 else x.to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)

    # every buffer at an alignment of its own
    at = iter(range(off, 10 ** 6, max(1, off)))
    x = [Padded(values(r), next(at) % 64) for r in rows]
    d = [Padded(values(drows), next(at) % 64) for _ in range(prob.n_dst)]
    g = [Padded(values(drows), next(at) % 64) for _ in range(prob.n_dst)]
    y = [Padded(values(r), next(at) % 64) for r in rows]
    a = [Padded(rng.standard_normal((r, hidden), dtype=np.float32), next(at) % 64) for r in rows]
    cut = lambda b: b.whole[b.at:b.at + b.n].copy().reshape(b.t.shape)                # noqa: E731
    T = lambda bs: [b.t for b in bs]                                                  # noqa: E731

    want_d, want_y, want_a = [cut(b) for b in d], [cut(b) for b in y], [cut(b) for b in a]
    prob.forward([cut(b) for b in x], want_d)
    (prob.backward_f32 if f32 else prob.backward_bf16)([cut(b) for b in g], want_y)
    prob.backward_accumulate([cut(b) for b in g], want_a)
    hp.hp_forward(plan, T(x), T(d))
    hp.hp_backward(plan, T(g), T(y))
    hp.hp_backward_accumulate(plan, T(g), T(a))
    torch.cuda.synchronize()
    for kind, bufs, want in (("forward", d, want_d), ("backward", y, want_y), ("accumulate", a, want_a)):
        for i, (b, w) in enumerate(zip(bufs, want)):
            b.check(w, (kind, i))
    for b, w in zip(d, want_d):
        b.whole[b.at:b.at + b.n] = w.reshape(-1)
    prob_zero = [w.view(np.uint32 if f32 else np.uint16).copy() for w in want_d]
    for j, z in enumerate(prob_zero):
        sb, _ = prob.forward_map(j)
        z[sb >= 0] = 0
    hp.hp_zero_image_rows(plan, T(d))
    text = [Padded(values(drows), next(at) % 64) for _ in range(prob.n_dst)]
    hp.hp_text_grads(plan, T(g), T(text))
    torch.cuda.synchronize()
    for j, (b, z) in enumerate(zip(d, prob_zero)):
        b.check(z, ("zero", j))
    for j, (b, t) in enumerate(zip(g, text)):
        want = cut(b)
        want[prob.forward_map(j)[0] >= 0] = 0
        t.check(want, ("text", j))
        b.check(cut(b), ("gradient", j))
    plan.close()


# hp_text_grads: one launch of runs, several, or (many short runs: more launches than the bytes are worth) a copy and
# a pass of zeros; no image at all; row-strided columns
@pytest.mark.parametrize("n_img,hidden,f32,sbh", [(0, 96, False, False), (0, 96, False, True), (3, 4096, False, True),
                                                  (257, 72, False, False), (257, 16384, True, False),
                                                  (300, 200, False, True)])
def test_text_gradients(n_img, hidden, f32, sbh):
    rng = np.random.default_rng(n_img)
    dst = wl.Grid(tp=2, row_order=wl.ROW_SBH if sbh else wl.ROW_BSH)
    samp = np.sort(rng.integers(0, 2, n_img)).astype(np.int32)
    start = np.concatenate([4 * np.arange(int((samp == b).sum())) for b in range(2)]).astype(np.int32)
    seq = 4 * max(1, n_img) + 2
    tm = wl.TokenMap(2, seq, hidden, samp, start, rng.integers(1, 4, n_img).astype(np.int32), None, int(f32))
    plan = hp.hp_plan_create(wl.Grid(), dst, tm)
    dt = torch.float32 if f32 else torch.bfloat16
    g = [torch.randn(2 * seq, hidden, device="cuda").to(dt) for _ in range(2)]
    out = [torch.full_like(t, 7.0) for t in g]
    keep = [t.clone() for t in g]
    for _ in range(2):                                      # the first call and one that finds the runs
        hp.hp_text_grads(plan, g, out)
    image = torch.zeros(2, seq, dtype=torch.bool)
    for b, s, n in zip(tm.img_sample, tm.img_start, tm.img_len):
        image[int(b), int(s):int(s) + int(n)] = True
    image = (image.t() if sbh else image).reshape(-1).cuda()
    for t, o, k in zip(g, out, keep):
        assert torch.equal(o, torch.where(image[:, None], torch.zeros_like(t), t)) and torch.equal(t, k)
    plan.close()


# many short runs: whole buffers are copied, whatever the row order, and their image rows zeroed; small ones through the
# memory-side cache, large ones (the last two) past it
@pytest.mark.parametrize("batch,seq,hidden,tp,f32,sbh", [(300, 20, 72, 2, False, True), (300, 20, 67, 3, True, True),
                                                         (513, 9, 64, 1, False, False), (1, 1500, 1001, 2, False, False),
                                                         (2, 33000, 2112, 1, False, True), (1, 66000, 2111, 1, False, False)])
def test_text_gradients_of_many_short_images(batch, seq, hidden, tp, f32, sbh):
    per = max(1, 600 // batch)
    samp = np.repeat(np.arange(batch), per).astype(np.int32)
    start = np.tile(np.arange(per) * (seq // per) + 1, batch).astype(np.int32)
    tm = wl.TokenMap(batch, seq, hidden, samp, start, np.full(len(samp), 1, np.int32), None, int(f32))
    plan = hp.hp_plan_create(wl.Grid(dp=2), wl.Grid(tp=tp, row_order=wl.ROW_SBH if sbh else wl.ROW_BSH), tm)
    dt = torch.float32 if f32 else torch.bfloat16
    g = [torch.randn(batch * seq, hidden, device="cuda").to(dt) for _ in range(tp)]
    out = [torch.full_like(t, 7.0) for t in g]
    keep = [t.clone() for t in g]
    hp.hp_text_grads(plan, g, out)
    image = torch.zeros(batch, seq, dtype=torch.bool)
    image[torch.from_numpy(samp).long(), torch.from_numpy(start).long()] = True
    image = (image.t() if sbh else image).reshape(-1).cuda()
    for t, o, k in zip(g, out, keep):
        assert torch.equal(o, torch.where(image[:, None], torch.zeros_like(t), t)) and torch.equal(t, k)
    plan.close()


# where a plan's tables go: with a launch's arguments or into device memory (the tree's levels and the last segments
# that fit: 1 level up to 16 segments, arguments full a little above 100)
@pytest.mark.parametrize("n_seg", [1, 16, 17, 32, 100, 104, 105, 106, 107, 108, 109, 110, 112, 130, 257])
def test_tables_in_the_arguments_and_in_device_memory(n_seg):
    rng = np.random.default_rng(n_seg)
    src, dst = wl.Grid(dp=1), wl.Grid(tp=2)
    seq, hidden = 4 * n_seg + 3, 72
    start = (4 * np.arange(n_seg)).astype(np.int32)
    tm = wl.TokenMap(1, seq, hidden, np.zeros(n_seg, np.int32), start, rng.integers(1, 4, n_seg).astype(np.int32))
    plan, prob = hp.hp_plan_create(src, dst, tm), oracle.Problem(src, dst, tm)
    assert plan.info.n_segments == n_seg and plan.info.on_device == 1
    bits = lambda n, s: wl.bf16_bits(wl.random_bf16((n, hidden), s))                  # noqa: E731
    rows, drows = prob.src_rows(), prob.dst_rows()
    x, d, g = [bits(r, 1) for r in rows], [bits(drows, 2 + j) for j in range(2)], [bits(drows, 4 + j) for j in range(2)]
    dev = lambda a: torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)     # noqa: E731
    back = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16)                # noqa: E731
    X, D, E, G = [dev(a) for a in x], [dev(a) for a in d], [dev(a) for a in d], [dev(a) for a in g]
    Y = [torch.zeros_like(t) for t in X]
    host = hp.hp_plan_create_host(src, dst, tm)
    hp.hp_forward(plan, X, D)
    hp.hp_forward_static(host, X, E)
    hp.hp_backward(plan, G, Y)
    plan.close()                                            # with its launches still queued
    torch.cuda.synchronize()
    y = [np.zeros_like(a) for a in x]
    prob.forward(x, d)
    prob.backward_bf16(g, y)
    for j in range(2):
        assert np.array_equal(back(D[j]), d[j]) and np.array_equal(back(E[j]), d[j])
    assert np.array_equal(back(Y[0]), y[0])
    with pytest.raises(hp.HpError):
        hp.hp_forward(host, X, D)                           # a host-only plan is refused, however small


@pytest.mark.parametrize("src_grad,text_grad,graph", [(True, False, False), (False, True, False), (True, True, True)])
def test_autograd_gives_only_the_gradients_that_are_wanted(src_grad, text_grad, graph):
    """Frozen text embeddings, a frozen encoder, and create_graph: the same values as with everything trained."""
    rng = np.random.default_rng(9)
    dst = wl.Grid(tp=2, cp=2)
    tm = wl.token_map_from_lens(rng, 2, 24, 40, [[5, 7], [9]])
    plan = hp.hp_plan_create(wl.Grid(dp=2), dst, tm)
    drows = plan.info.dst_rows_per_buf
    new = lambda r, s: wl.random_bf16((r, 40), s, "cuda")                             # noqa: E731

    def grads(src_on, text_on, create):
        x = [new(r, i).requires_grad_(src_on) for i, r in enumerate(plan.src_rows())]
        t = [new(drows, 10 + j).requires_grad_(text_on) for j in range(4)]
        w = [new(drows, 20 + j) for j in range(4)]
        outs = hp.boundary_transform(plan, x, [a.clone() for a in t])
        g = torch.autograd.grad(outs, x * src_on + t * text_on, w, create_graph=create)
        return list(g[:len(x)]) if src_on else [], list(g[len(x):]) if src_on else list(g)

    want_x, want_t = grads(True, True, False)
    got_x, got_t = grads(src_grad, text_grad, graph)
    assert len(got_x) == len(want_x) * src_grad and len(got_t) == len(want_t) * text_grad
    assert all(torch.equal(a, b) for a, b in zip(got_x, want_x)) and all(torch.equal(a, b) for a, b in zip(got_t, want_t))
    plan.close()


@pytest.mark.parametrize("tp_src,src_on,text_on,maps", [(1, True, True, 1), (2, True, True, 1), (3, True, False, 2),
                                                        (1, False, True, 1)])
def test_second_derivatives(tp_src, src_on, text_on, maps):
    """Gradients taken with create_graph, differentiated again, against autograd of the definition in 64 bits: every copy of a
    source rank has the gradient of its rows, text embeddings that of theirs, and none from under the image rows."""
    rng = np.random.default_rng(tp_src)
    src, dst = wl.Grid(tp=tp_src, dp=2), wl.Grid(tp=2, cp=2, cp_split=wl.CP_ZIGZAG, row_order=wl.ROW_SBH)
    tms = [wl.token_map_from_lens(rng, 2, 24, 9, [[5, 7], [9]]) for _ in range(maps)]
    for tm in tms:
        tm.dtype = wl.DT_F32
    plan = hp.hp_plan_create_batched(src, dst, tms) if maps > 1 else hp.hp_plan_create(src, dst, tms[0])
    probs = [oracle.Problem(src, dst, tm) for tm in tms]
    rows, drows, n_dst = plan.src_rows(), plan.info.dst_rows_per_buf, plan.info.n_dst_bufs
    new = lambda r: torch.from_numpy(rng.standard_normal((r, 9)))                     # noqa: E731
    x, t, u, v = [new(r) for r in rows], [new(drows) for _ in range(n_dst)], [new(r) for r in rows], [new(drows) for _ in range(n_dst)]
    per_src, per_dst = len(rows) // maps, n_dst // maps

    # the definition: for each destination buffer the source buffer and row of its image rows
    where = []
    for m, prob in enumerate(probs):
        for j in range(per_dst):
            sb, sr = (torch.from_numpy(np.asarray(a)).long() for a in prob.forward_map(j))
            where.append((torch.where(sb >= 0, sb + m * per_src, sb), sr))

    def definition(xs, ts):
        outs = []
        for (sb, sr), b in zip(where, ts):
            o = [xs[int(s)][int(r)] if s >= 0 else b[k] for k, (s, r) in enumerate(zip(sb, sr))]
            outs.append(torch.stack(o))
        return outs

    def second(xs, ts, us, vs, transform, ref):
        xs = [a.clone().requires_grad_(src_on) for a in xs]
        ts = [a.clone().requires_grad_(text_on) for a in ts]
        read = [xs[i - i % tp_src] for i in range(len(xs))] if ref else xs             # forward reads copy 0
        outs = transform(read, [a.clone() for a in ts])
        loss = sum((o ** 3).sum() * (1 + k) for k, o in enumerate(outs))
        wanted = xs * src_on + ts * text_on
        if ref:                                                                        # ... and every copy gets its gradient
            wanted = [xs[i - i % tp_src] for i in range(len(xs))] * src_on + ts * text_on
        g = torch.autograd.grad(loss, wanted, create_graph=True)
        s = sum((a * (b ** 2 + b)).sum() for a, b in zip(us * src_on + vs * text_on, g))
        leaders = xs[::tp_src] * src_on + ts * text_on
        plain = torch.autograd.grad(sum(b.sum() + b.t().reshape(-1)[::2].sum() for b in g), leaders, retain_graph=True)
        return [a.detach() for a in g], [*plain, *torch.autograd.grad(s, leaders)]  # cotangents expanded, strided, plain

    x = [x[i - i % tp_src] for i in range(len(x))]          # the copies of a rank hold the same rows
    want_g, want_s = second(x, t, u, v, definition, True)
    dev = lambda a: [b.float().cuda() for b in a]                                      # noqa: E731
    got_g, got_s = second(dev(x), dev(t), dev(u), dev(v), lambda a, b: hp.boundary_transform(plan, a, b), False)
    # all sums are of a few dozen terms in binary32: 2^-24 each, measured against the largest value
    for got, want in ((got_g, want_g), (got_s, want_s)):
        assert len(got) == len(want)
        for a, b in zip(got, want):
            scale = float(b.abs().max()) if b.numel() else 1.0
            assert torch.allclose(a.cpu().double(), b, rtol=0, atol=1e-5 * scale)
    plan.close()


def test_plans_made_while_the_last_ones_still_run():
    """Plans with tables in device memory, each used on one of two busy streams and dropped at once: every launch reads
    its own plan's tables."""
    dst, hidden, n_seg = wl.Grid(tp=2), 72, 300
    seq = 4 * n_seg
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    busy = torch.randn(4096, 4096, device="cuda")
    x = wl.random_bf16((2 * seq, hidden), 3, "cuda")
    outs, maps = [], []
    torch.cuda.synchronize()
    for i in range(24):
        rng = np.random.default_rng(i)
        start = np.sort(rng.choice(np.arange(0, seq, 4), n_seg - i, replace=False)).astype(np.int32)
        tm = wl.TokenMap(1, seq, hidden, np.zeros(n_seg - i, np.int32), start, rng.integers(1, 4, n_seg - i).astype(np.int32))
        st = streams[i % 2]
        with torch.cuda.stream(st):
            busy @ busy
            out = [torch.zeros(seq, hidden, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
            plan = hp.hp_plan_create(wl.Grid(), dst, tm)
            hp.hp_forward(plan, [x], out, st)
            plan.close()
        outs.append(out)
        maps.append(tm)
    torch.cuda.synchronize()
    for out, tm in zip(outs, maps):
        pos = np.concatenate([np.arange(s, s + n) for s, n in zip(tm.img_start, tm.img_len)])
        want = torch.zeros(seq, hidden, dtype=torch.bfloat16, device="cuda")
        want[torch.from_numpy(pos).cuda()] = x[:len(pos)]
        assert torch.equal(out[0], want) and torch.equal(out[1], want)
