"""Stage 2 by sorting networks, against the oracle, bit for bit: up to 64 winners behind one slot per bucket (composites), and up to 256 of 1024 bf16
candidates behind queues (a positive value and its index in one word), with too few positive candidates for that, ties, and k at the blocks' edges."""
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


def _rows(m, n, seed, dtype):
    x = workloads.normal_rows(m, n, seed=seed)
    x[1] = (x[1] * 2).round() / 2
    x[2] = -x[2].abs()                                             # nothing positive
    x[3] = torch.where(torch.arange(n) % 1000 == 7, 1.0, -1.0)     # few positive, ties
    x[4] = x[4].sort().values
    x[5] = torch.where(x[5] > 0, 0.0, -0.0)                        # zeros of either sign
    x[6, n // 2:] = -float("inf")
    x[7] = workloads.special_values(1, n, seed=seed)[0]
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _check(x, k, b, k_b, dtype):
    print(dtype, tuple(x.shape), k, b, k_b, atk.plan_describe(*x.shape, k, b, k_b, atk.ATK_F32 if dtype == "f32" else atk.ATK_BF16), flush=True)
    vals, idx = atk.approx_topk(x.cuda(), k, b, k_b)
    torch.cuda.synchronize()
    ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8)
    assert np.array_equal(idx.cpu().numpy(), oi)
    got = vals.cpu()
    assert np.array_equal(got.numpy().view(np.uint32), ov.view(np.uint32)) if dtype == "f32" else np.array_equal(got.view(torch.int16).numpy().view(np.uint16), ov)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n, b, spec", [(8192, 128, ""), (8192, 256, ""), (8192, 512, ""), (8192, 1024, ""), (16384, 64, "BO=0"), (65536, 256, "BO=0"),
                                        (65536, 512, "BO=0"), (65536, 1024, "BO=0"), (1 << 18, 256, "BO=0"), (8000, 200, "BO=0"), (13200, 264, "BO=0"),
                                        (65536, 1024, "BO=0,T=256,LN=1")])
def test_one_slot(n, b, spec, dtype, plan_override):
    plan_override((spec + "," if spec else "") + "WV=0")
    x = _rows(8, n, n + b, dtype)
    for k in (1, 2, 33, 63, 64):
        if k < b:
            _check(x, k, b, 1, dtype)


# workgroups of 320, 384 and 448 lanes: more buckets than four wavefronts sort, where the lanes see too few matrix rows for bins
@pytest.mark.parametrize("dtype, b", [("f32", 1024), ("f32", 1028), ("f32", 1100), ("f32", 1280), ("f32", 1536), ("f32", 1788), ("f32", 1792), ("bf16", 1024),
                                      ("bf16", 1032), ("bf16", 1040), ("bf16", 1152), ("bf16", 1536)])
def test_more_buckets_than_networks_hold(dtype, b):
    for L in (8, 16):
        n = L * b
        x = _rows(8, n, n + b, dtype)
        x[6] = torch.where(torch.arange(n) % b >= min(1024, b - 4), x[6].abs() + 10.0, x[6])  # winners in the last buckets alone
        for k in (1, 33, 64):
            _check(x, k, b, 1, dtype)
            g = x.cuda()
            vals, idx = torch.empty((8, k), dtype=x.dtype, device="cuda"), torch.empty((8, k), dtype=torch.int32, device="cuda")
            assert atk.approx_topk_noalloc_raw(g.data_ptr(), 8, n, k, b, 1, atk.ATK_F32 if dtype == "f32" else atk.ATK_BF16, vals.data_ptr(), idx.data_ptr(),
                                               torch.cuda.current_stream().cuda_stream) == 0
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy(), oracle.approx_topk(workloads.as_numpy_bits(x), k, b, 1, threads=8)[1])


def test_advised_buckets():
    b, k_b = atk.advise(1, 9216, 24, atk.ATK_F32, 0.9)[:2]
    _check(_rows(8, 9216, 24, "f32")[:1], 24, b, k_b, "f32")


@pytest.mark.parametrize("n", [50000, 128256, 131072, 131080])
@pytest.mark.parametrize("b, k_b", [(512, 2), (64, 4), (250, 4), (128, 8), (60, 16), (100, 3)])
def test_words(n, b, k_b):
    x = _rows(8, n, n + b, "bf16")
    for k in (20, 64, 65, 200, 255, 256):
        if k_b <= k < b * k_b:
            _check(x, k, b, k_b, "bf16")
