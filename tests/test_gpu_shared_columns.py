"""f32 queues of eight and sixteen slots over wide bucket layouts, which four lanes of a workgroup share where the rows would be split, against the
oracle, bit for bit: without Stage 2 and with it, in the same launch (one split and several) and apart, fewer slots used than there are, odd lengths,
buckets that do not divide them, rows off the 16-byte boundaries, workgroups halved for their exchange area, and few rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_04358_amd as atk
from paper_2412_04358_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [(128, 1 << 18, 1024, 1024, 8, 0), (128, 1 << 18, 8192, 1024, 8, 0), (100, 300001, 1000, 777, 8, 0), (130, 1 << 18, 700, 1026, 5, 0),
                                  (128, 1 << 20, 1024, 1024, 16, 0), (100, 300001, 1000, 777, 8, 3), (169, 131072, 100, 215, 8, 0),
                                  (88, 104995, 64, 139, 8, 1), (322, 1 << 18, 4944, 412, 12, 0), (128, 1 << 17, 474, 158, 12, 0), (3, 85417, 462, 231, 8, 2)])
def test_shared(case):
    assert torch.cuda.is_available(), "this test needs the MI355X"
    m, n, k, b, k_b, shift = case
    plan = atk.plan_describe(m, n, k, b, k_b, atk.ATK_F32)
    print(case, plan, flush=True)
    assert " P=4 " in plan, plan
    x = workloads.normal_rows(m, n, seed=b + k_b)
    x[1] = x[1].sort().values
    x[2] = workloads.few_levels(1, n, levels=3, seed=1)[0]
    buf = torch.empty(x.numel() + shift, device="cuda")
    g = buf[shift:].view(x.shape)
    g.copy_(x)
    vals, idx = atk.approx_topk(g, k, b, k_b)
    torch.cuda.synchronize()
    rows = [0, 1, 2, m // 2, m - 1]
    ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x[rows].contiguous()), k, b, k_b, threads=8)
    assert np.array_equal(idx[rows].cpu().numpy(), oi)
    assert np.array_equal(vals[rows].cpu().numpy().view(np.uint32), ov.view(np.uint32))
