"""exact_topk of rows that one workgroup holds in registers, and Stage 2 over (value, index) pairs, against the oracle:
bit for bit, at the edges of the instances' sizes and on rows that take each way through the kernel."""
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


def _check(x, k, shift=0):
    print("exact %s %s k=%d shift=%d" % (tuple(x.shape), x.dtype, k, shift), flush=True)
    g = x.cuda()
    if shift:
        buf = torch.empty(x.numel() + shift, dtype=x.dtype, device="cuda")
        g = buf[shift:].view(x.shape)
        g.copy_(x)
    vals, idx = atk.exact_topk(g, k)
    torch.cuda.synchronize()
    ov, oi = oracle.exact_topk(workloads.as_numpy_bits(x), k, threads=8)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(_bits(vals), ov.view(np.uint32) if ov.dtype == np.float32 else ov)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("m", [2, 300])
def test_sizes(m, dtype):
    """Around one vector, one wavefront, and the largest row of each workgroup size; k from 1 to the whole row."""
    ve = 4 if dtype == "f32" else 8
    for n in (1, ve - 1, ve + 1, 64 * ve, 128 * ve + 1, 512 * ve, 512 * ve + 3, 1024 * ve - 1, 2048 * ve, 2048 * ve + ve):
        for k in sorted({1, min(n, 5), max(1, n // 16), max(1, n // 4), n}):
            if m * n < 3e6 or k <= n // 4:
                _check(workloads.normal_rows(m, n, seed=n + k, dtype=dtype), k)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_largest_rows(dtype):
    ve = 4 if dtype == "f32" else 8
    n = 1024 * 16 * ve
    for k in (1, 64, 1000, 16384, 16385):
        _check(workloads.normal_rows(2, n, seed=k, dtype=dtype), k)
    for rows in (n - 1, n - ve + 1, n + 1):  # one vector short of what fits off the 16-byte boundaries, and beyond it
        _check(workloads.normal_rows(3, rows, seed=rows, dtype=dtype), 300, shift=1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_ways_through(dtype):
    """Rows whose first guess fails, whose bins are crowded (ties, values around zero, an outlier), masked rows."""
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    for n in (1000, 8192, 40000):
        base = workloads.normal_rows(3, n, seed=n)
        rows = [workloads.few_levels(3, n, levels=3, seed=n, dtype=dtype), workloads.special_values(3, n, seed=n, dtype=dtype),
                base.sort(dim=1)[0].to(t), base.sort(dim=1, descending=True)[0].to(t), torch.zeros(3, n, dtype=t),
                (-base.abs() - 1.0).to(t), torch.relu(base).to(t)]
        masked = base.clone()
        masked[:, n // 20:] = float("-inf")
        outlier = base.clone()
        outlier[:, n // 2] = 3.0e38
        blocks = base.clone()
        blocks[:, : n // 2] += 100.0
        rows += [masked.to(t), outlier.to(t), blocks.to(t)]
        for x in rows:
            for k in (7, 200, n // 4):
                _check(x, k)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pairs(dtype):
    """Stage 2 over more candidates than the fused kernels select from: lists of (value, index) pairs."""
    for (m, n, k, b, k_b) in [(3, 65536, 4096, 4096, 2), (2, 40000, 100, 4099, 1), (300, 16384, 1025, 4104, 1), (2, 70000, 5000, 2050, 4),
                              (2, 131072, 8192, 16384, 1), (2, 65536, 10, 10007, 1)]:
        x = workloads.normal_rows(m, n, seed=b, dtype=dtype)
        print("pairs", m, n, k, b, k_b, dtype, flush=True)
        vals, idx = atk.approx_topk(x.cuda(), k, b, k_b)
        torch.cuda.synchronize()
        ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8)
        assert np.array_equal(idx.cpu().numpy(), oi)
        assert np.array_equal(_bits(vals), ov.view(np.uint32) if ov.dtype == np.float32 else ov)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_in_parts(dtype):
    """Rows shared out between workgroups: uneven parts, rows off the 16-byte boundaries, parts unlike each other, ties."""
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    ve = 4 if dtype == "f32" else 8
    for (m, n, k) in [(1, 12288 * ve, 64), (2, 12289 * ve + 1, 1), (128, 16384 * ve, 100), (3, 16385 * ve, 1000), (2, 8192 * ve * 5 + 7, 300),
                      (300, 16384 * ve + 3, 10), (1, 1 << 21, 1024), (2, 8192 * 8 * 64 + 1 if dtype == "bf16" else 8192 * 4 * 64 + 1, 33)]:
        if m * n < 2.5e7:
            _check(workloads.normal_rows(m, n, seed=n % 1000 + k, dtype=dtype), k, shift=1 if n % 2 else 0)
    n = 20000 * ve
    base = workloads.normal_rows(2, n, seed=3)
    blocks = base.clone()
    blocks[:, n // 3: n // 3 + 2000] += 50.0
    for x in (base.sort(dim=1)[0], base.sort(dim=1, descending=True)[0], blocks, torch.zeros(2, n), torch.relu(base - 5.0)):
        for k in (1, 90, 800):
            _check(x.to(t), k)
    _check(workloads.few_levels(2, n, levels=3, seed=9, dtype=dtype), 500)
    _check(workloads.special_values(2, n, seed=9, dtype=dtype), 500)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(3, 1 << 18, 64), (2, 1 << 20, 1000), (70, 1 << 18, 20), (5, 200003, 300)])
def test_parts_unlike_each_other(shape, dtype):
    """Rows whose parts hold more or fewer of the winners than their share: masked, with a trend, in one place, neighbours that go
    together, ties at every place of the range."""
    m, n, k = shape
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    base = workloads.normal_rows(m, n, seed=n % 977)
    rows = [base + torch.linspace(0.0, 6.0, n), base.sort(dim=1)[0], torch.full((m, n), 0.3), torch.full((m, n), -0.0)]
    for at in (slice(0, n // 33), slice(0, n // 2), slice(n - n // 20, n), slice(n // 4, n), slice(0, n - k // 2)):
        masked = base.clone()
        masked[:, at] = float("-inf")
        rows.append(masked)
    stripes = base.clone()
    stripes[:, (torch.arange(n) // 4096) % 2 == 0] = float("-inf")
    block = base.clone()
    block[:, n // 3: n // 3 + n // 64] += 50.0
    spikes = torch.zeros(m, n)
    spikes[:, 5] = 2.0
    spikes[:, (n * 7) // 9] = 1.0
    lagged = torch.nn.functional.avg_pool1d(base.unsqueeze(1), 65, 1, 32).squeeze(1) * 8.0
    rows += [stripes, block, spikes, lagged, torch.relu(base - 1.5), (base * 100.0).round(), torch.randint(0, 3, (m, n)).float()]
    for x in rows:
        _check(x.to(t).contiguous(), k, shift=n % 2)
