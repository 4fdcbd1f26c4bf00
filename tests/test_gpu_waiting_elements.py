"""Eight-slot queues with pooled floors, whose elements wait beside the queue until a second one comes: rows on which every element enters, none
after the first, or ties decide, with lanes that stop early and with queues shorter than the slots, against the oracle, bit for bit."""
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


@pytest.fixture
def plan_override():
    yield atk.set_plan_override
    atk.set_plan_override(None)


def _rows(n):
    x = workloads.normal_rows(1, n, seed=n)
    return torch.cat([x, x.sort(dim=1).values, x.sort(dim=1, descending=True).values, workloads.few_levels(1, n, levels=1, seed=1),
                      workloads.few_levels(1, n, levels=3, seed=2), workloads.special_values(1, n, seed=3)]).contiguous()


@pytest.mark.parametrize("spec", ["P=8,RF=8", "P=8,RF=1,S=1", "P=32,RF=8,T=256", "P=2,RF=4,S=2"])
@pytest.mark.parametrize("case", [(65536, 16, 8), (65538, 14, 5), (40000, 8, 7), (1 << 18, 64, 8)])
def test_waiting(case, spec, plan_override):
    n, b, k_b = case
    x = _rows(n)
    plan_override(spec)
    for k in (b * k_b, 40):
        plan = atk.plan_describe(x.shape[0], n, k, b, k_b, atk.ATK_F32)
        print(n, k, b, k_b, plan, flush=True)
        assert " refresh=0" not in plan
        vals, idx = atk.approx_topk(x.cuda(), k, b, k_b)
        torch.cuda.synchronize()
        ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8)
        assert np.array_equal(idx.cpu().numpy(), oi)
        assert np.array_equal(vals.cpu().numpy().view(np.uint32), ov.view(np.uint32))
