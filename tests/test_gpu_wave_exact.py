"""exact_topk of short bf16 rows, a wavefront each, against the oracle, bit for bit: rows without order, in order, of ties, of one value, masked in
part, without a positive element; every compiled size, and k at the edges of the lists."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_04358_amd as atk
from paper_2412_04358_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu_and_lib():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    atk.load_library()


def _rows(n, seed):
    g = torch.Generator().manual_seed(seed)
    z = torch.randn((12, n), generator=g)
    u = torch.rand((12, n), generator=g)
    x = z.clone()
    x[1] = (z[1] * 1.5).round()
    x[2] = 1.0                                                    # ties from the first element to the last
    x[3] = torch.where(u[3] < 0.5, 1.0, -1.0)
    x[4] = z[4].sort().values
    x[5] = z[5].sort(descending=True).values
    x[6, n // 3:] = -float("inf")                                 # masked from a third on
    x[7] = torch.where(u[7] < 0.99, -float("inf"), z[7])          # fewer numbers than winners, then ties of -inf
    x[8] = -z[8].abs() - 0.5                                      # no positive element
    x[9] = torch.where(u[9] < 0.3, torch.where(u[9] < 0.15, 0.0, -0.0), -z[9].abs())  # winners that are zeros of either sign
    x[10] = torch.where(u[10] < 0.001, float("inf"), z[10] * 1e-39)                   # denormals
    x[11] = torch.where(torch.arange(n) % 64 < 2, 100.0 + z[11], z[11])               # the largest in a few lanes
    return x.to(torch.bfloat16)


def _check(x, k, out=None):
    vals, idx = atk.exact_topk(x.cuda(), k, out=out)
    torch.cuda.synchronize()
    ov, oi = oracle.exact_topk(workloads.as_numpy_bits(x), k)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(vals.cpu().view(torch.int16).numpy().view(np.uint16), ov)


@pytest.mark.parametrize("n", [8, 64, 504, 512, 520, 1024, 1032, 1544, 2048, 2056, 4096, 4104, 6144, 6152, 7000, 8184, 8192])
def test_sizes(n, plan_override):
    plan_override("WV=1")
    x = _rows(n, n)
    for k in (1, 3, 63, 64, 65, 100, 120, 128, 129, 256, 257, 512, 513, 700, 896):
        if k <= n:
            print(n, k, flush=True)
            _check(x, k)


@pytest.mark.parametrize("m, n, k", [(1100, 8192, 512), (1024, 6144, 129), (3, 2048, 300), (5, 4096, 64), (2500, 1024, 200), (4, 512, 512),
                                     # either side of the lists that a workgroup a row is quicker with
                                     (3, 1536, 513), (3, 1544, 513), (3, 2048, 512), (1030, 2304, 513), (1030, 2312, 513), (1030, 4104, 575),
                                     (1030, 4104, 576), (2049, 8192, 256), (2049, 8192, 384), (2049, 8192, 385), (2048, 6152, 300)])
def test_chosen(m, n, k):
    _check(_rows(n, k).repeat(-(-m // 12), 1)[:m].contiguous(), k)


def test_addresses(plan_override):
    """Outputs off the 16-byte boundaries; x off them is another plan's."""
    plan_override("WV=1")
    n, k = 4096, 256
    x = _rows(n, 1)
    vals = torch.empty(12 * k + 1, dtype=torch.bfloat16, device="cuda")[1:].view(12, k)
    idx = torch.empty(12 * k + 1, dtype=torch.int32, device="cuda")[1:].view(12, k)
    _check(x, k, out=(vals, idx))
    store = torch.zeros(12 * n + 1, dtype=torch.bfloat16, device="cuda")
    store[1:].view(12, n).copy_(x)
    got = atk.exact_topk(store[1:].view(12, n), k)
    assert torch.equal(got[1], idx) and torch.equal(got[0].view(torch.int16), vals.view(torch.int16))
