"""One survivor per bucket and no Stage 2 (b = k) on rows whose columns several workgroups share out, the last of them fewer than the others: running maxima that
meet in LDS, with helpers and a finisher too, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_04358_amd as atk
from paper_2412_04358_amd import workloads


def _plan(m, n, b, dtype):
    return {k: int(v) for k, v in (kv.split("=") for kv in atk.plan_describe(m, n, b, b, 1, atk.ATK_F32 if dtype == "f32" else atk.ATK_BF16).split())}


# (rows, matrix rows, buckets, whether the specialised kernels take them, helpers)
CASES = [("f32", 159, 56, 456, 1, 0), ("f32", 1, 4, 104, 1, 0), ("f32", 64, 4, 776, 1, 0), ("f32", 3, 500, 216, 1, 1), ("f32", 8, 128, 488, 1, 1),
         ("bf16", 159, 56, 1312, 1, 0), ("bf16", 1, 4, 208, 1, 0), ("bf16", 2, 500, 432, 1, 1), ("bf16", 1, 128, 1456, 1, 1),
         ("bf16", 1, 128, 130, 0, 0), ("bf16", 159, 128, 186, 0, 0)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype, m, L, b, lean, helpers", CASES)
def test_narrow_last_block(dtype, m, L, b, lean, helpers):
    n = L * b
    p = _plan(m, n, b, dtype)
    print(dtype, m, n, b, p, flush=True)
    assert p["colblocks"] > 1 and b % (p["Gw"] * p["V"]) and p["lean"] == lean and (p["helpers"] > 0) == bool(helpers)
    large = torch.full((512, 8192), 1e30, device="cuda")
    for x in (workloads.normal_rows(m, n, seed=b, dtype=dtype), -workloads.normal_rows(m, n, seed=L, dtype=dtype).abs(), workloads.special_values(m, n, seed=b, dtype=dtype)):
        ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), b, b, 1, threads=8)
        g = x.cuda()
        for _ in range(3):
            atk.approx_topk(large, 64, 512, 1)  # (leaves large values in every CU's LDS)
            vals, idx = atk.approx_topk(g, b, b, 1)
            torch.cuda.synchronize()
            assert np.array_equal(idx.cpu().numpy(), oi)
            got = vals.cpu()
            assert np.array_equal(got.numpy().view(np.uint32), ov.view(np.uint32)) if dtype == "f32" else np.array_equal(got.view(torch.int16).numpy().view(np.uint16), ov)
