"""The boundary transform as one differentiable PyTorch operation.

The paper's boundary communicator is an autograd-aware operation: its forward
materialises the source module's activation in the destination layout and its
backward applies the reverse transform (Method, paragraph on boundary edges).
This module only strings the library's calls together for torch.autograd -
every tensor element is still moved by the HIP kernels behind hp_forward,
hp_backward and hp_text_grads:

    outs = boundary_transform(plan, src_bufs, text_bufs)

`text_bufs` are the destination buffers already holding the text embeddings;
they are modified in place (the image-token rows are overwritten) and returned.
Backward gives, for every source buffer, the TP-summed gradient of its rows (all
TP copies of a source rank receive the same gradient) and, for every text
buffer, the incoming gradient with the image-token rows set to zero.  With
create_graph these are differentiable in turn, to any order.
"""
from __future__ import annotations

from typing import List, Sequence

import torch

from .binding import Plan


# torch's own names for the current device and its current stream's handle; not part of its interface, so that
# another torch may be without them
_get_device = getattr(torch._C, "_cuda_getDevice", None)
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _current_stream() -> int:
    """The handle of torch's current stream.  torch.cuda.current_stream() makes an object around it first, 2.7 us of a
    pass that is bound by the host (123 MB in 16 buffers: 112 us)."""
    if _raw_stream is None or _get_device is None:
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(_get_device())


class _BoundaryTransform(torch.autograd.Function):
    @staticmethod
    def forward(ctx, plan: Plan, n_src: int, *bufs):
        src, dst = list(bufs[:n_src]), list(bufs[n_src:])
        stream = _current_stream()
        plan.forward([t.detach() if t is not None else None for t in src], [t.detach() for t in dst], stream)
        ctx.plan, ctx.n_src = plan, n_src
        ctx.src_meta = [(tuple(t.shape), t.dtype, t.device) for t in src]
        ctx.mark_dirty(*dst)
        return tuple(dst)

    @staticmethod
    def backward(ctx, *grad_dst):
        n = ctx.n_src
        want = any(ctx.needs_input_grad[2:2 + n]), any(ctx.needs_input_grad[2 + n:])
        if torch.is_grad_enabled():                         # create_graph: differentiable in turn
            got = _BoundaryGrads.apply(ctx.plan, ctx.src_meta, want, *grad_dst)
        else:
            got = _grads(ctx.plan, ctx.src_meta, want, grad_dst)
        k = n if want[0] else 0
        return (None, None, *(got[:k] or (None,) * n), *(got[k:] or (None,) * len(grad_dst)))


def _grads(plan: Plan, src_meta, want, grad_dst) -> tuple:
    """The source gradients and the text gradients, each if they are wanted, in one tuple."""
    stream = _current_stream()
    grads = [g.contiguous() for g in grad_dst]
    src_grads: List[torch.Tensor] = []
    if want[0]:
        src_grads = [torch.empty(shape, dtype=dtype, device=device) for shape, dtype, device in src_meta]
        plan.backward(grads, src_grads, stream)
    # gradient with respect to the text embeddings: the rows forward replaced carry none
    text_grads: List[torch.Tensor] = []
    if want[1]:
        text_grads = [torch.empty_like(g) for g in grads]
        plan.text_grads(grads, text_grads, stream)
    return (*src_grads, *text_grads)


class _BoundaryGrads(torch.autograd.Function):
    """_grads as a function of the destination gradients, in which it is linear: its derivative carries cotangents of the
    source gradients to the image rows and cotangents of the text gradients to the others, as the transform itself does."""

    @staticmethod
    def forward(ctx, plan: Plan, src_meta, want, *grad_dst):
        ctx.plan, ctx.src_meta, ctx.want = plan, src_meta, want
        return _grads(plan, src_meta, want, [g.detach() for g in grad_dst])

    @staticmethod
    def backward(ctx, *h):
        plan, (want_src, want_text) = ctx.plan, ctx.want
        n = len(ctx.src_meta) if want_src else 0
        if not want_src:                                    # the image rows get nothing
            return (None, None, None, *_BoundaryGrads.apply(plan, ctx.src_meta, ctx.want, *h))
        if want_text:
            dst = [t.clone(memory_format=torch.contiguous_format) for t in h[n:]]
        else:
            dst = [h[0].new_zeros(plan.info.dst_rows_per_buf, plan.hidden) for _ in range(plan.info.n_dst_bufs)]
        # every copy of a source rank received the same sum: their cotangents add up, in the copy that forward reads
        src = [t.contiguous() for t in h[:n]]
        i = 0
        for copies in plan.src_copies():
            if copies > 1:
                src[i] = torch.stack(src[i:i + copies]).float().sum(0).to(src[i].dtype)
                src[i + 1:i + copies] = [t.detach() for t in src[i + 1:i + copies]]
            i += copies
        return (None, None, None, *boundary_transform(plan, src, dst))


def boundary_transform(plan: Plan, src_bufs: Sequence[torch.Tensor], text_bufs: Sequence[torch.Tensor]):
    """Differentiable hp_forward: returns the destination buffers (the same
    tensors as `text_bufs`, modified in place) as a tuple.  Every source buffer
    must be a tensor (empty ranks: a [0, hidden] tensor).  Runs on torch's
    current stream."""
    if len(src_bufs) != plan.info.n_src_bufs or len(text_bufs) != plan.info.n_dst_bufs:
        raise ValueError("wrong number of buffers for this plan")
    return _BoundaryTransform.apply(plan, len(src_bufs), *src_bufs, *text_bufs)
