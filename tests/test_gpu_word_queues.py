"""Queues of eight and sixteen slots that hold a float's own bits and its row's number as a double: zeros of either sign, the smallest and largest
floats, infinities and ties, in rows that end inside a batch or start inside a load, against the oracle, bit for bit."""
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


def _rows(n, dtype):
    g = torch.Generator().manual_seed(n)
    # the smallest denormal, the two floats on either side of a double's smallest exponent, the largest float, the smallest normal one
    bits = [0x0, 0x80000000, 0x1, 0x80000001, 0x000FFFFF, 0x00100000, 0x800FFFFF, 0x80100000, 0x7F7FFFFF, 0xFF7FFFFF, 0x7F800000, 0xFF800000,
            0x00800000, 0x80800000, 0x3F800000, 0xBF800000]
    vals = torch.from_numpy(np.array(bits, dtype=np.uint32).view(np.float32).copy())
    x = torch.empty((4, n))
    x[0] = vals[torch.randint(len(bits), (n,), generator=g)]
    x[1] = vals[torch.randint(8, (n,), generator=g)]                                # around zero
    x[2] = -torch.rand((n,), generator=g) - 0.5                                     # negative, with a zero here and there
    x[2][torch.rand((n,), generator=g) < 0.05] = 0.0
    x[2][torch.rand((n,), generator=g) < 0.05] = -0.0
    x[3] = torch.where(torch.rand((n,), generator=g) < 0.8, -float("inf"), -1.0)  # buckets whose queues end in ties of -inf
    if dtype == "bf16":
        x = (x.view(torch.int32) & -65536).view(torch.float32).to(torch.bfloat16)
    return x.contiguous()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
# (k_b, matrix rows): whole batches, one row more, one less than two batches, queues that no batch fills, long lanes
@pytest.mark.parametrize("k_b, rows", [(8, 32), (8, 33), (8, 15), (5, 9), (8, 8), (7, 200), (16, 64), (16, 47), (9, 17)])
@pytest.mark.parametrize("b, spec", [(256, "PK=0,S=1"), (258, "PK=0,S=1,P=1"), (64, "PK=0,S=3"), (16, "PK=0,P=8,RF=1,S=1")])
def test_words(dtype, k_b, rows, b, spec, plan_override):
    plan_override(spec)
    code = atk.ATK_F32 if dtype == "f32" else atk.ATK_BF16
    for n in (rows * b, rows * b + b // 2 + 1):
        x = _rows(n, dtype)
        for k in (b * k_b, b * k_b // 3):
            print(dtype, n, k, b, k_b, atk.plan_describe(4, n, k, b, k_b, code), flush=True)
            vals, idx = atk.approx_topk(x.cuda(), k, b, k_b)
            torch.cuda.synchronize()
            ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8)
            assert np.array_equal(idx.cpu().numpy(), oi)
            got = vals.cpu().view(torch.int32 if dtype == "f32" else torch.int16).numpy()
            assert np.array_equal(got.view(ov.dtype if dtype == "bf16" else np.uint32), ov if dtype == "bf16" else ov.view(np.uint32))
