"""approx_topk of short bf16 rows that one wavefront takes alone, its candidates sorted in registers, against the oracle, bit for bit; and, on the
CPU, that a plan of this kind is only made where the kernel's assumptions hold."""
import random

import numpy as np
import pytest
import torch

import oracle
import paper_2412_04358_amd as atk
from paper_2412_04358_amd import workloads


def _plan(m, n, k, b, k_b):
    return dict(kv.split("=") for kv in atk.plan_describe(m, n, k, b, k_b, atk.ATK_BF16).split())


def _rows(m, n, seed):
    """Rows without order, of ties, of zeros of either sign among negative values, of infinities, rising and falling ones."""
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((m, n), generator=g)
    for r in range(m):
        kind = r % 6
        if kind == 1:
            x[r] = (x[r] * 1.5).round()
        elif kind == 2:
            u = torch.rand((n,), generator=g)
            x[r] = -x[r].abs() - 0.1
            x[r][u < 0.04] = 0.0
            x[r][u < 0.02] = -0.0
        elif kind == 3:
            x[r][torch.rand((n,), generator=g) < 0.7] = -float("inf")
            x[r][::97] = float("inf")
        elif kind == 4:
            x[r] = x[r].sort().values
        elif kind == 5:
            x[r] = x[r].sort(descending=True).values
    return x.to(torch.bfloat16)


def _check(x, k, b, k_b, out=None):
    vals, idx = atk.approx_topk(x.cuda() if not x.is_cuda else x, k, b, k_b, out=out)
    torch.cuda.synchronize()
    ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x.cpu()), k, b, k_b, threads=8)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(vals.cpu().view(torch.int16).numpy().view(np.uint16), ov)


# every (columns per lane, column groups, slots) that is compiled, at both ends of its bucket counts
LAYOUTS = [(b, k_b) for b, kbs in ((66, (2, 3, 8)), (128, (2, 4, 7)), (132, (1, 2, 8)), (256, (1, 3, 8)), (264, (1, 2, 4)), (512, (1, 2, 3)),
                                   (520, (1, 2)), (1024, (1, 2))) for k_b in kbs]


@pytest.mark.gpu
@pytest.mark.parametrize("b, k_b", LAYOUTS)
def test_layouts(b, k_b):
    """One batch of matrix rows, parts of batches, and a ragged last row; k at the edges of the sorted blocks' sizes, and odd."""
    v = 2 if b <= 128 else 4 if b <= 256 else 8
    for n in {b * k_b, b * 16, b * 17 + v, b * 9 - v, b * 40 + b - v}:
        if n < b * k_b or n > 12288:
            continue
        x = _rows(7, n, n + k_b)
        for k in {k_b, 63, 64, 65, 128, 129, b * k_b // 4, b * k_b // 2, b * k_b // 2 + 1, b * k_b - 1}:
            if k_b <= k < b * k_b and k <= 1024:
                print(n, k, b, k_b, flush=True)
                assert int(_plan(7, n, k, b, k_b)["wave"]) > 0
                _check(x, k, b, k_b)


# loads of one and of two elements, in every number of groups and with every length of queues that is compiled
NARROW = [(b, k_b) for b, kbs in ((65, (2, 3, 8)), (127, (2, 4, 7)), (129, (1, 2, 4)), (130, (1, 2, 4)), (254, (1, 2, 3)), (255, (1, 2, 3)), (257, (1, 2)),
                                  (258, (1, 2)), (510, (1, 2)), (511, (1, 2)), (513, (1, 2)), (514, (1, 2)), (1022, (1, 2)), (1023, (1, 2))) for k_b in kbs]


@pytest.mark.gpu
@pytest.mark.parametrize("b, k_b", NARROW)
def test_narrow_loads(b, k_b):
    try:
        atk.set_plan_override("WV=1")
        v = 2 - b % 2
        for n in {b * k_b, b * 3 + 1, b * 16, b * 17 + v, b * 33 - v}:
            if n < b * k_b or n > 12288:
                continue
            x = _rows(7, n, n + k_b)
            for k in {k_b, 64, 65, b * k_b // 2 + 1, b * k_b - 1}:
                if k_b <= k < b * k_b and k <= 1024:
                    print(n, k, b, k_b, flush=True)
                    p = _plan(7, n, k, b, k_b)
                    assert int(p["wave"]) > 0 and int(p["V"]) == (2 if b % 2 == 0 and n % 2 == 0 else 1)
                    _check(x, k, b, k_b)
    finally:
        atk.set_plan_override(None)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(2049, 2048, 100, 128, 2), (1030, 16384, 500, 512, 1), (2048, 65536, 700, 512, 4)])
def test_many_rows(case):
    m, n, k, b, k_b = case
    assert int(_plan(m, n, k, b, k_b)["wave"]) > 0
    _check(_rows(m, n, 3), k, b, k_b)


@pytest.mark.gpu
def test_addresses():
    """x off the 16-byte boundaries is another plan's; outputs off them are written element by element."""
    m, n, k, b, k_b = 6, 4096, 256, 512, 2
    store = torch.zeros(m * n + 1, dtype=torch.bfloat16, device="cuda")
    x = store[1:].view(m, n)
    x.copy_(_rows(m, n, 5))
    _check(x, k, b, k_b)
    vals = torch.empty(m * k + 1, dtype=torch.bfloat16, device="cuda")[1:].view(m, k)
    idx = torch.empty(m * k + 1, dtype=torch.int32, device="cuda")[1:].view(m, k)
    _check(_rows(m, n, 5), k, b, k_b, out=(vals, idx))


def test_rows_too_long_for_their_buckets():
    """Few buckets leave the lanes long columns: those rows are a workgroup's."""
    for n, b, wave in ((7260, 66, True), (7262, 66, False), (12276, 66, False), (12288, 112, True), (16384, 82, True), (16384, 80, False)):
        assert (int(_plan(2048, n, 64, b, 2)["wave"]) > 0) == wave, (n, b)


@pytest.mark.parametrize("spec", ["T=256", "S=2", "V=4", "P=2", "PK=0", "TS=0", "LN=0", "LM=0", "HF=0", "HF=1", "HQ=40", "HT=512", "SL=128", "MH=0", "MH=2", "BO=0", "RF=0", "RF=4"])
def test_a_key_that_names_another_plan_is_obeyed(spec, plan_override):
    assert int(_plan(64, 8192, 100, 256, 1)["wave"]) > 0
    plan_override(spec)
    assert int(_plan(64, 8192, 100, 256, 1)["wave"]) == 0
    plan_override(spec + ",WV=1")
    assert int(_plan(64, 8192, 100, 256, 1)["wave"]) > 0


def test_plans_fit_the_kernel():
    rng = random.Random(1)
    seen = 0
    for _ in range(4000):
        b = rng.randint(1, 1300)
        if rng.random() < 0.7:
            b -= b % rng.choice((2, 4, 8))
        n = rng.randint(max(b, 1), rng.choice((4000, 13000, 70000)))
        if rng.random() < 0.7:
            n -= n % 8
        if b < 1 or n < b:
            continue
        k_b = rng.randint(1, min(16, n // b))
        if b * k_b < 2:
            continue
        k, m = rng.randint(k_b, b * k_b), rng.choice((1, 100, 1024, 5000))
        p = _plan(m, n, k, b, k_b)
        r = int(p["wave"])
        assert (p["stage2"] == "3") == (r > 0)
        if not r:
            continue
        seen += 1
        v, kb = int(p["V"]), int(p["KB"])
        groups = 1  # (a power of two)
        while 64 * v * groups < b:
            groups *= 2
        assert b % v == 0 and n % v == 0 and groups <= (16 // v if v < 4 else 2 if v == 8 else 1)
        assert kb >= k_b and v * groups * kb <= 32
        words = v * groups * kb
        assert words % r == 0 and 64 * r >= k and r * 8 >= words and k < b * k_b and n <= 65536
        assert int(p["scratch_bytes"]) == 0
    assert seen > 300
