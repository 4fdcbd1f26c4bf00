"""Calls on plain tensors, which an extension module marshals, against the same calls with `out`, which binding.py does itself; and what is no plain call:
subclasses, modes, arguments that are no integers, tensors and parameters that are refused."""
import threading
import warnings

import numpy as np
import pytest
import torch
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2412_04358_amd as atk
from paper_2412_04358_amd import binding, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu_and_lib():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    x = workloads.normal_rows(2, 1024, seed=1).cuda()
    atk.exact_topk(x, 4)  # (the first call loads the module)
    assert binding._plain is not None


def _same(got, want):
    assert isinstance(got, tuple) and type(got[0]) is torch.Tensor and type(got[1]) is torch.Tensor
    assert got[0].dtype == want[0].dtype and got[1].dtype == torch.int32 and got[0].device == want[0].device
    assert torch.equal(got[1], want[1]) and torch.equal(got[0], want[0]) and not got[0].requires_grad


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_plain(dtype):
    x = workloads.normal_rows(5, 4096, seed=2, dtype=dtype).cuda()
    out = (torch.empty((5, 64), dtype=x.dtype, device="cuda"), torch.empty((5, 64), dtype=torch.int32, device="cuda"))
    for call in (lambda y, **kw: atk.approx_topk(y, 64, 128, 1, **kw), lambda y, **kw: atk.approx_topk(y, 64, 32, 2, assignment=atk.ATK_INTERLEAVED, **kw),
                 lambda y, **kw: atk.approx_topk(y, k=64, b=256, k_b=1, assignment=atk.ATK_CONTIGUOUS, **kw), lambda y, **kw: atk.exact_topk(y, 64, **kw)):
        want = tuple(t.clone() for t in call(x, out=out))
        _same(call(x), want)
        with torch.inference_mode():
            _same(call(x), want)
        _same(call(torch.nn.Parameter(x)), want)
        _same(call(x.clone().requires_grad_()), want)
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            got = call(x)
        s.synchronize()
        _same(got, want)
        got = [None] * 4

        def run(i):
            got[i] = call(x)
            torch.cuda.synchronize()

        threads = [threading.Thread(target=run, args=(i,)) for i in range(4)]
        [t.start() for t in threads]
        [t.join() for t in threads]
        for g in got:
            _same(g, want)


@pytest.mark.parametrize("why", ["missing", "damaged", "another torch"])
def test_without_the_module(why, tmp_path, monkeypatch):
    """Calls need the library alone: with `out` the module is not even asked for, without a warning says that it cannot be used."""
    x = workloads.normal_rows(3, 4096, seed=4).cuda()
    want = atk.approx_topk(x, 64, 128, 1), atk.exact_topk(x, 64)
    if why == "another torch":
        monkeypatch.setattr(torch, "__version__", "0.0.1")
    else:
        path = tmp_path / "_atk_torch.so"
        if why == "damaged":
            path.write_bytes(b"no library")
        monkeypatch.setattr(binding, "_TORCH_PATH", str(path))
    monkeypatch.setattr(binding, "_plain", None)
    out = (torch.empty((3, 64), device="cuda"), torch.empty((3, 64), dtype=torch.int32, device="cuda"))
    _same(atk.approx_topk(x, 64, 128, 1, out=out), want[0])
    _same(atk.exact_topk(x, 64, out=out), want[1])
    assert binding._plain is None
    with pytest.warns(RuntimeWarning, match="cannot be used"):
        _same(atk.exact_topk(x, 64), want[1])
    assert binding._plain is False
    with warnings.catch_warnings():
        warnings.simplefilter("error")  # (once is enough)
        _same(atk.approx_topk(x, 64, 128, 1), want[0])
    with pytest.raises(binding.ApproxTopkError):
        atk.exact_topk(x, 0)


def test_not_plain():
    x = workloads.normal_rows(3, 2048, seed=3).cuda()
    want = atk.exact_topk(x, 10)
    _same(tuple(t.as_subclass(torch.Tensor) for t in atk.exact_topk(x.as_subclass(type("T", (torch.Tensor,), {})), 10)), want)
    seen = []

    class Functions(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    class Dispatch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    for mode in (Functions, Dispatch):
        seen.clear()
        with mode():
            got = atk.exact_topk(x, 10)
        assert seen
        _same(got, want)
    _same(atk.exact_topk(x, True), atk.exact_topk(x, 1))
    for bad in (lambda: atk.exact_topk(x, 0), lambda: atk.exact_topk(x, 2049), lambda: atk.approx_topk(x, 64, 8, 4), lambda: atk.approx_topk(x, 64, 64, 1, assignment=7),
                lambda: atk.approx_topk(x, 64, 1 << 62, 1)):
        with pytest.raises(binding.ApproxTopkError):
            bad()
    for bad in (x.t(), x[:, ::2], x[0], x.cpu()):
        with pytest.raises(ValueError):
            atk.exact_topk(bad, 4)
    with pytest.raises(TypeError):
        atk.exact_topk(x.half(), 4)
    with pytest.raises(Exception):
        atk.exact_topk(x, 1 << 70)
    with pytest.raises(Exception):
        atk.exact_topk(x, 4.0)
    with pytest.raises(RuntimeError):
        atk.exact_topk(x, -1)
    assert np.array_equal(atk.exact_topk(x, 10)[1].cpu().numpy(), want[1].cpu().numpy())
