"""exact_topk of bf16 rows in parts, marked as packed keys, against the oracle, bit for bit: rows off the vectors' boundaries, negative rows, rows
unlike themselves, ties (which a part cuts before it passes them on), every workgroup size.  k at the edges of the plans for 9 rows: groups of
twice as many maxima from 257, 513 and 1025 on, a second bound that cuts the parts' lists from 121 to 337 on (817 with three parts), and 1600 near
the largest k of twelve and more parts."""
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
    x = torch.randn((9, n), generator=g)
    u = torch.rand((n,), generator=g)
    x[1] = x[1] - 6.0                                             # all of it negative
    x[2] = torch.where(u < 0.0005, x[2].abs(), -x[2].abs() - 1.0)  # few positive elements
    x[3] = (x[3] * 2).round()
    x[4] = x[4].sort().values
    x[5, n // 3:] = -float("inf")
    x[6] = torch.where(u < 0.2, 0.0, torch.where(u < 0.4, -0.0, -x[6].abs()))
    x[7] = 1.0
    x[8] = workloads.special_values(1, n, seed=seed)[0]
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("spec", ["", "T=512", "T=256", "S=3", "S=7,T=1024"])
@pytest.mark.parametrize("n", [100000, 100003, 128256, 131071, 150001])
def test_parts(n, spec, plan_override):
    plan_override(spec)
    x = _rows(n, n)
    for k in (1, 63, 64, 65, 200, 256, 257, 513, 816, 817, 1025, 1600):
        print(n, k, spec, flush=True)
        vals, idx = atk.exact_topk(x.cuda(), k)
        torch.cuda.synchronize()
        ov, oi = oracle.exact_topk(workloads.as_numpy_bits(x), k)
        assert np.array_equal(idx.cpu().numpy(), oi)
        assert np.array_equal(vals.cpu().view(torch.int16).numpy().view(np.uint16), ov)
