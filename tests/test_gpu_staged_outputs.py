"""Direct plans (every bucket's queue is the output) whose outputs go through LDS, against the oracle, bit for bit: whole wavefronts, and the last one's part."""
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m, n, b, k_b", [(3, 16384, 512, 8), (2, 16384, 256, 16), (130, 8192, 1024, 8), (2, 40000, 1250, 8), (3, 20000, 625, 16), (5, 4096, 130, 8)])
def test_staged_outputs(m, n, b, k_b, dtype):
    x = workloads.normal_rows(m, n, seed=b, dtype=dtype)
    for off in (0, 1):  # outputs on the 16-byte boundaries and off them
        vals = torch.empty(m * b * k_b + off, dtype=x.dtype, device="cuda")[off:].view(m, b * k_b)
        idx = torch.empty(m * b * k_b + off, dtype=torch.int32, device="cuda")[off:].view(m, b * k_b)
        atk.approx_topk(x.cuda(), b * k_b, b, k_b, out=(vals, idx))
        torch.cuda.synchronize()
        ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), b * k_b, b, k_b, threads=8)
        assert np.array_equal(idx.cpu().numpy(), oi)
        got = vals.cpu()
        assert np.array_equal(got.numpy().view(np.uint32), ov.view(np.uint32)) if dtype == "f32" else np.array_equal(got.view(torch.int16).numpy().view(np.uint16), ov)
