"""Queues of one 32-bit word per slot (bf16, two slots and more) against the oracle, bit for bit: rows whose every survivor is a zero of
either sign, subnormals next to zero, as many matrix rows as are packed, and one more."""
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


def _check(x, k, b, k_b):
    print("%s k=%d b=%d k_b=%d [%s]" % (tuple(x.shape), k, b, k_b, atk.plan_describe(*x.shape, k, b, k_b, atk.ATK_BF16)), flush=True)
    vals, idx = atk.approx_topk(x.cuda(), k, b, k_b)
    torch.cuda.synchronize()
    ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(vals.cpu().view(torch.int16).numpy().view(np.uint16), ov)


def _zeros(m, n, seed):
    """Below zero but for a few zeros of both signs and subnormals, in stretches longer and shorter than a queue."""
    g = torch.Generator().manual_seed(seed)
    x = -torch.rand((m, n), generator=g) - 0.5
    u = torch.rand((m, n), generator=g)
    x[u < 0.02] = 0.0
    x[u < 0.01] = -0.0
    x[u < 0.0005] = 1e-39
    x[u < 0.0003] = -1e-39
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("k_b", [2, 3, 4, 8, 16])
@pytest.mark.parametrize("n", [4096, 8191, 70001])
def test_zeros(n, k_b):
    for b in (32, 33):
        _check(_zeros(3, n, n + b), min(40, b * k_b), b, k_b)


@pytest.mark.parametrize("v", [1, 2, 4, 8])
@pytest.mark.parametrize("rows", [65533, 65534])
def test_last_row_number(rows, v, plan_override):
    """One lane to a column group and one split: `rows` matrix rows in it, the most that pack and one more, a ragged row after them and, in rows
    that start off a load's boundary, one whole row more; the winners are in the last of these and tie with others at the start."""
    b = 64 * v
    plan_override("V=%d,S=1,T=64" % v)
    n = rows * b + b - 1
    for k_b in (2, 4, 8) if v <= 2 else (2, 4) if v == 4 else (2,):
        p = dict(kv.split("=") for kv in atk.plan_describe(3, n, b * k_b, b, k_b, atk.ATK_BF16).split())
        assert (p["V"], p["P"], p["S"], p["rows_per_split"], p["packed"]) == (str(v), "1", "1", str(rows), "1" if rows < 65534 else "0"), p
        x = torch.full((3, n), -1.0, dtype=torch.bfloat16)
        x[0] = workloads.few_levels(1, n, levels=3, seed=v, dtype="bf16")[0]
        x[1, -b * k_b :: 3] = 1.0
        x[1, : b * 5] = torch.arange(b * 5).remainder(2).to(torch.bfloat16)
        x[2, -b:] = 2.0
        x[2, -2 * b : -b] = torch.arange(b).remainder(5).to(torch.bfloat16)
        _check(x, b * k_b, b, k_b)


@pytest.mark.parametrize("v", [1, 2, 4, 8])
@pytest.mark.parametrize("rows", [65024, 65535, 65537])
def test_most_matrix_rows(rows, v, plan_override):
    """One split of some 65024 matrix rows, a number of rounds of its lanes, and one round more: packed and unpacked queues; the winners at either
    end and ties between them."""
    b = 8
    plan_override("V=%d,S=1" % v)
    n = rows * b + 3
    assert " packed=%d " % (rows <= 65024) in atk.plan_describe(2, n, 16, b, 2, atk.ATK_BF16)  # (a split is whole rounds of its lanes)
    x = workloads.few_levels(2, n, levels=3, seed=v, dtype="bf16")
    x[1] = -1.0
    x[1, -5:] = 1.0
    x[1, :9] = 1.0
    _check(x, 16, b, 2)
    _check(x, 32, b, 4)
