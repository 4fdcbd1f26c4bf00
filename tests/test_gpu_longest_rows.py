"""Rows of nearly 2^31 elements in one bucket, the longest that the column indices number: every lane's scan ends within a few batches of 2^31,
where numbers of 32 bits for the rows to come would wrap.  A few winners lie in a constant row, at both ends and where workgroups' shares meet."""
import pytest
import torch

import paper_2412_04358_amd as atk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("assignment", [atk.ATK_INTERLEAVED, atk.ATK_CONTIGUOUS])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_one_bucket(dtype, assignment):
    assert torch.cuda.is_available(), "this test needs the MI355X"
    n = (1 << 31) - 1
    at = [0, 1, 511, (1 << 29) + 7, (1 << 30) - 1, 1 << 30, n - 9000, n - 4097, n - 513, n - 300, n - 257, n - 129, n - 64, n - 17, n - 2, n - 1]
    value = [3.0, 9.0, 5.0, 8.0, 2.0, 5.0, 7.0, 5.0, 4.0, 1.0, 6.0, 9.0, 5.0, 0.5, 9.0, 10.0]
    order = sorted(range(len(at)), key=lambda i: (-value[i], at[i]))
    x = torch.full((1, n), -1.0, device="cuda", dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    x[0, torch.tensor(at, device="cuda")] = torch.tensor(value, device="cuda").to(x.dtype)
    for k_b in (1, 2, 4, 5, 8, 16):
        print(dtype, assignment, k_b, atk.plan_describe(1, n, k_b, 1, k_b, atk.ATK_F32 if dtype == "f32" else atk.ATK_BF16, assignment), flush=True)
        vals, idx = atk.approx_topk(x, k_b, 1, k_b, assignment=assignment)
        torch.cuda.synchronize()
        assert idx[0].tolist() == [at[i] for i in order[:k_b]]
        assert vals[0].float().tolist() == [value[i] for i in order[:k_b]]
