"""Stage 2 as a launch of its own over (value, index) pairs, chosen by the planner or forced, and the queues of distinct
words in front of it, against the oracle, bit for bit."""
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


def _bits(t):
    t = t.cpu().contiguous()
    return t.numpy().view(np.uint32) if t.dtype == torch.float32 else t.view(torch.int16).numpy().view(np.uint16)


def _check(x, k, b, k_b, assignment=None, shift=0):
    g = x.cuda()
    if shift:
        buf = torch.empty(x.numel() + shift, dtype=x.dtype, device="cuda")
        g = buf[shift:].view(x.shape)
        g.copy_(x)
    print("approx %s %s k=%d b=%d k_b=%d shift=%d" % (tuple(x.shape), x.dtype, k, b, k_b, shift), flush=True)
    vals, idx = atk.approx_topk(g, k, b, k_b, assignment=assignment)
    torch.cuda.synchronize()
    ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8,
                                assignment=oracle.CONTIGUOUS if assignment == atk.ATK_CONTIGUOUS else oracle.INTERLEAVED)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(_bits(vals), ov.view(np.uint32) if ov.dtype == np.float32 else ov)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(4, 8192, 1024, 2048, 1), (40, 8192, 512, 1024, 1), (1, 65536, 1024, 512, 8), (2, 65536, 64, 4096, 1),
                                  (1100, 4096, 64, 512, 2), (1030, 2048, 300, 128, 8), (3, 20000, 2000, 683, 4), (2, 16384, 1024, 1024, 2)])
def test_chosen(case, dtype, plan_override):
    """The pairs' launch; bf16 rows that one wavefront would take alone by their own plan, off the 16-byte boundaries, and kept off it."""
    m, n, k, b, k_b = case
    x = workloads.normal_rows(m, n, seed=b, dtype=dtype)
    plan = atk.plan_describe(m, n, k, b, k_b, atk.ATK_F32 if dtype == "f32" else atk.ATK_BF16)
    if " wave=0 " not in plan:
        assert dtype == "bf16" and " stage2=3 " in plan, plan
        _check(x, k, b, k_b)
        _check(x, k, b, k_b, shift=1)
        plan_override("WV=0")
        plan = atk.plan_describe(m, n, k, b, k_b, atk.ATK_BF16)
    assert " stage2=2 " in plan and " wave=0 " in plan and " scratch_bytes=0 " not in plan, plan
    _check(x, k, b, k_b)
    if m <= 40:
        _check(workloads.few_levels(m, n, levels=3, seed=b, dtype=dtype), k, b, k_b)
        _check(workloads.special_values(m, n, seed=b, dtype=dtype), k, b, k_b)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_forced(dtype):
    """Lists of every size against the selection in the same launch, rows off the 16-byte boundaries, contiguous buckets."""
    try:
        for spec in ("TS=1", "TS=0"):
            atk.set_plan_override(spec)
            for (m, n, k, b, k_b) in [(3, 1000, 1, 2, 1), (2, 4097, 10, 33, 3), (5, 8192, 64, 65, 1), (2, 70001, 100, 511, 2), (300, 4096, 100, 128, 4)]:
                _check(workloads.normal_rows(m, n, seed=b, dtype=dtype), k, b, k_b, shift=1 if n % 2 else 0)
                _check(workloads.normal_rows(m, n, seed=b, dtype=dtype), k, b, k_b, assignment=atk.ATK_CONTIGUOUS)
    finally:
        atk.set_plan_override(None)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k_b", [5, 8, 9, 16])
def test_queues_of_words(k_b, dtype):
    """Infinities, signed zeros, denormals, ties and buckets that end inside a batch of rows; k_b below the number of slots."""
    for (m, n, b) in [(3, 4096, 64), (2, 5003, 61), (2, 70000, 100), (130, 65536, 1024), (1, 1 << 18, 256)]:
        if n // b >= k_b:
            xs = [workloads.normal_rows(m, n, seed=b + k_b, dtype=dtype)]
            if m <= 3:
                xs += [workloads.special_values(m, n, seed=b, dtype=dtype), workloads.few_levels(m, n, levels=2, seed=b, dtype=dtype),
                       torch.full((m, n), float("-inf"), dtype=xs[0].dtype), torch.full((m, n), float("inf"), dtype=xs[0].dtype)]
            for x in xs:
                _check(x, b * k_b, b, k_b)
                if m <= 3:
                    _check(x, max(k_b, b * k_b // 3), b, k_b)
