"""The marshalling extension: what it takes is what the way through Python takes, and what it leaves is still reported."""
import os
import subprocess
import sys
import warnings

import numpy as np
import pytest
import torch

import paper_2605_27678_amd as hp
from paper_2605_27678_amd import binding
from paper_2605_27678_amd import workloads as wl


def make(host_only):
    tm = wl.token_map_from_lens(np.random.default_rng(1), 2, 16, 8, [[3], [4, 2]])
    args = wl.Grid(dp=2), wl.Grid(tp=2), tm
    return hp.hp_plan_create_host(*args) if host_only else hp.hp_plan_create(*args)


def buffers(plan, device):
    new = lambda r: torch.randn(r, 8, device=device).to(torch.bfloat16)               # noqa: E731
    return [new(r) for r in plan.src_rows()], [new(plan.info.dst_rows_per_buf) for _ in range(plan.info.n_dst_bufs)]


def test_host_buffers_and_foreign_objects_take_the_way_through_python():
    plan = make(True)
    src, dst = buffers(plan, "cpu")
    for a, b in ((src, dst), (tuple(src), dst), (iter(src), dst), (src, [1, 2])):
        assert plan._call("hp_forward", binding.SRC, a, binding.DST, b, None) is False
    with pytest.raises(ValueError, match="contiguous CUDA tensor"):
        hp.hp_forward(plan, src, dst)
    with pytest.raises(ValueError, match="wrong number"):
        hp.hp_forward(plan, src[:1], dst)
    plan.close()
    with pytest.raises(ValueError):
        hp.hp_forward(plan, src, dst)


def test_the_binding_goes_on_without_the_extension(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_PKG", str(tmp_path))
    monkeypatch.setattr(binding, "_marshal", None)
    plan = make(True)
    src, dst = buffers(plan, "cpu")
    with pytest.warns(RuntimeWarning, match="hp_marshal.so is not used"):
        with pytest.raises(ValueError, match="contiguous CUDA tensor"):
            hp.hp_forward(plan, src, dst)
    with warnings.catch_warnings():
        warnings.simplefilter("error")                      # said once
        assert plan._call("hp_forward", binding.SRC, src, binding.DST, dst, None) is False


def test_an_extension_for_another_torch_is_not_used(monkeypatch):
    monkeypatch.setattr(binding, "_marshal", None)
    monkeypatch.setattr(torch, "__version__", "0.0")
    with pytest.warns(RuntimeWarning, match="built for torch"):
        assert make(True)._call("hp_forward", binding.SRC, [], binding.DST, [], None) is False


@pytest.mark.parametrize("gone", ["torch", "g++", "headers"])
def test_the_library_builds_without_the_extension(monkeypatch, tmp_path, gone):
    from paper_2605_27678_amd import build
    lib, ext, ran = tmp_path / "libhp.so", tmp_path / "hp_marshal.so", []
    ext.write_text("an older one")
    monkeypatch.setattr(build, "LIB_PATH", str(lib))
    monkeypatch.setattr(build, "MARSHAL_PATH", str(ext))
    if gone == "torch":
        monkeypatch.setitem(sys.modules, "torch", None)

    def run(cmd, **kw):
        ran.append(os.path.basename(cmd[0]))
        if cmd[0] == "g++" and gone == "g++":
            raise FileNotFoundError("g++")
        if cmd[0] != "g++":
            lib.write_text("built")
        return subprocess.CompletedProcess(cmd, int(cmd[0] == "g++"), "", "no headers")

    monkeypatch.setattr(build.subprocess, "run", run)
    assert build.build_library() == str(lib) and lib.exists() and not ext.exists()
    assert ran[-1] == "hipcc" and ("g++" in ran) == (gone != "torch")


@pytest.mark.parametrize("name", ["_raw_stream", "_get_device"])
def test_the_current_stream_without_torchs_own_names(monkeypatch, name):
    from types import SimpleNamespace
    from paper_2605_27678_amd import autograd
    monkeypatch.setattr(autograd, name, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=77))
    assert autograd._current_stream() == 77


@pytest.mark.gpu
def test_the_current_stream_is_torchs():
    from paper_2605_27678_amd import autograd
    for stream in (torch.cuda.Stream(), torch.cuda.default_stream()):
        with torch.cuda.stream(stream):
            assert autograd._current_stream() == stream.cuda_stream == torch.cuda.current_stream().cuda_stream


@pytest.mark.gpu
def test_device_buffers():
    plan, host = make(False), make(True)
    src, dst = buffers(plan, "cuda")
    want = [t.clone() for t in dst]
    ps, pd = plan.pointer_arrays(src, want)
    plan.forward_raw(ps, pd)
    st = torch.cuda.Stream()
    for s in (None, torch.cuda.current_stream(), torch.cuda.current_stream().cuda_stream, st, st.cuda_stream):
        for kind in (list, tuple):
            got = [torch.where(w == w, t, t) for t, w in zip(dst, want)]
            torch.cuda.synchronize()
            assert plan._call("hp_forward", binding.SRC, kind(src), binding.DST, kind(got), s)
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(got, want))
    p = [torch.nn.Parameter(t) for t in src]
    assert plan._call("hp_forward", binding.SRC, p, binding.DST, dst, None)

    class Sub(torch.Tensor):
        pass
    sub = [t.as_subclass(Sub) for t in src]
    assert plan._call("hp_forward", binding.SRC, sub, binding.DST, dst, None) is False
    hp.hp_forward(plan, sub, dst)
    bad = [dst[0].t(), dst[0][:3], dst[0].float(), dst[0].cpu()]
    for b in bad:
        with pytest.raises(ValueError, match=r"dst\[0\]"):
            hp.hp_forward(plan, src, [b] + dst[1:])
    with pytest.raises(hp.HpError) as e:
        hp.hp_forward(plan, src, [None] + dst[1:])
    assert e.value.code == binding.HP_EINVAL
    with pytest.raises(hp.HpError) as e:
        hp.hp_forward(host, src, dst)
    assert e.value.code == binding.HP_ESTATE
    with pytest.raises(ValueError, match="src"):
        hp.hp_backward_accumulate(plan, dst, src)           # bf16 where binary32 accumulators belong
    torch.cuda.synchronize()
    plan.close()
    with pytest.raises(hp.HpError):
        hp.hp_forward(plan, src, dst)
