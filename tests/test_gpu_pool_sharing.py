"""approx_topk calls whose Stage 2 runs in a launch of its own, over pairs in the library's scratch, from several threads and
streams and under graph capture: the same results as from one stream, against the oracle, bit for bit."""
import threading

import numpy as np
import pytest
import torch

import oracle
import paper_2412_04358_amd as atk
from paper_2412_04358_amd import workloads

pytestmark = pytest.mark.gpu

# (m, n, k, b, k_b): Stage 2 apart by the planner's choice
_CALLS = [(4, 8192, 1024, 2048, 1), (2, 65536, 64, 4096, 1), (1100, 4096, 512, 512, 2), (128, 65536, 1024, 512, 8)]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu_and_lib():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    atk.load_library()


def _expected(x, k, b, k_b):
    v, i = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8)
    return torch.from_numpy(np.ascontiguousarray(v)).cuda(), torch.from_numpy(np.ascontiguousarray(i)).cuda()


def _cases():
    for at, (m, n, k, b, k_b) in enumerate(_CALLS):
        assert " stage2=2 " in atk.plan_describe(m, n, k, b, k_b) + " "
        x = workloads.normal_rows(m, n, seed=50 + at)
        yield x.cuda(), (k, b, k_b), _expected(x, k, b, k_b)


def test_threads_with_streams_of_their_own():
    cases = list(_cases())
    torch.cuda.synchronize()
    wrong, errors = [], []

    def work(at):
        try:
            x, args, (ev, ei) = cases[at]
            with torch.cuda.stream(torch.cuda.Stream()) as _:
                outs = [atk.approx_topk(x, *args) for _ in range(40)]
                torch.cuda.current_stream().synchronize()
            wrong.extend(at for v, i in outs if not (torch.equal(i, ei) and torch.equal(v, ev)))
        except Exception as e:  # noqa: BLE001 (reported below)
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(at,)) for at in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors and not wrong, (errors, wrong)


def test_streams_in_turn():
    cases = list(_cases())
    streams = [torch.cuda.Stream() for _ in cases]
    torch.cuda.synchronize()
    outs = []
    for _ in range(10):
        for at, (x, args, _e) in enumerate(cases):
            with torch.cuda.stream(streams[at]):
                outs.append((at, atk.approx_topk(x, *args)))
    torch.cuda.synchronize()
    for at, (v, i) in outs:
        assert torch.equal(i, cases[at][2][1]) and torch.equal(v, cases[at][2][0]), at


def test_captured_calls_keep_no_address_of_the_scratch():
    """Replays of a captured call after calls that let the scratch grow, and eager work in between."""
    (x, args, _e), (m, n) = next(_cases()), _CALLS[0][:2]
    other = workloads.normal_rows(m, n, seed=99)
    inputs = [(x, _expected(x.cpu(), *args)), (other.cuda(), _expected(other, *args))]
    xin = x.clone()
    out = (torch.empty((m, args[0]), device="cuda"), torch.empty((m, args[0]), dtype=torch.int32, device="cuda"))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(g, stream=side):
        atk.approx_topk(xin, *args, out=out)
    for rep in range(4):
        src, (ev, ei) = inputs[rep % 2]
        xin.copy_(src)
        out[0].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[1], ei) and torch.equal(out[0], ev), rep
        # (more scratch than any call of this module before it, a little more each time)
        big = workloads.normal_rows(64 << rep, 65536, seed=7).cuda()
        atk.approx_topk(big, 4096, 4096, 2)
        torch.cuda.synchronize()
