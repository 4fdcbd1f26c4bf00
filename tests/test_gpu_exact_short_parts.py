"""exact_topk of f32 rows that one workgroup holds and that are shared out between workgroups, on both sides of the lines in length and in rows, and for k
up to where one row after another goes back to one workgroup, against the oracle."""
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


@pytest.mark.parametrize("m, n", [(1, 49152), (3, 50001), (128, 49152), (2, 65533), (2, 65535), (1, 65536), (129, 49155)])
def test_either_side(m, n):
    x = torch.cat([workloads.normal_rows(m, n, seed=n, dtype="f32"), workloads.special_values(1, n, seed=m)])
    x[0, n // 2:] = -float("inf")
    want = oracle.exact_topk(workloads.as_numpy_bits(x), 2000)
    for k in (699, 700, 701, 1000, 2000):
        print(m, n, k, flush=True)
        vals, idx = atk.exact_topk(x.cuda(), k)
        torch.cuda.synchronize()
        assert np.array_equal(idx.cpu().numpy(), want[1][:, :k])
        assert np.array_equal(vals.cpu().numpy().view(np.uint32), want[0].view(np.uint32)[:, :k])
