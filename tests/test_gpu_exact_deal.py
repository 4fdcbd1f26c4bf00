"""exact_topk of long rows with many winners (elements dealt to bins), against the oracle, bit for bit: sizes at the edges of the
chunks and of what the sample allows, and rows that the sample misjudges or whose bins a workgroup cannot hold."""
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
def test_sizes(dtype):
    """n around whole chunks of 16384 and off the 16-byte boundaries; k from 64 sampled winners to over half the row."""
    for (m, n, k, shift) in [(2, 131080, 16385, 0), (1, 9 * 16384, 40000, 0), (3, 9 * 16384 + 1, 30000, 0), (2, 9 * 16384 - 3, 30000, 1),
                             (1, 1 << 20, 1 << 18, 0), (1, 1 << 21, 1 << 19, 0), (1, 1 << 20, (1 << 11) + 1, 0), (70, 140000, 20000, 0),
                             (2, 150001, 89999, 0), (2, 150001, 90002, 0)]:
        _check(workloads.normal_rows(m, n, seed=n % 1001 + k, dtype=dtype), k, shift)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_unlike_their_samples(dtype):
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    n = 200000
    base = workloads.normal_rows(2, n, seed=3)
    narrow = base.clone()
    narrow[:, 777: 777 + 20000] = 2.0 + 1e-3 * base[:, :20000]  # one place with most of the winners: bins past what LDS holds
    spikes = base.clone()
    spikes[:, :: 997] *= 1e18
    masked = base.clone()
    masked[:, n // 10:] = float("-inf")
    half = base.clone()
    half[:, : n // 3] += 50.0
    for x in (base.sort(dim=1)[0], base.sort(dim=1, descending=True)[0], narrow, spikes, masked, half, torch.relu(base), torch.zeros(2, n),
              (base * 64.0).round(), -base.abs()):
        _check(x.to(t), 30000)
    _check(workloads.few_levels(2, n, levels=3, seed=9, dtype=dtype), 50000)
    _check(workloads.special_values(2, n, seed=9, dtype=dtype), 50000)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [200000, 1 << 18, 1 << 20])
def test_elements_above_the_sampled_ones(n, dtype):
    """Winners above every sampled element: masked and rising rows, a few spikes over a long run of one value."""
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    base = workloads.normal_rows(2, n, seed=n % 1001)
    rows = [base.sort(dim=1)[0]]
    for part in (4, 2):
        for fill in (float("-inf"), 0.0):
            masked = base.clone()
            masked[:, : n // part] = fill
            rows.append(masked)
    for at in ([5], [n - 7], [3, n // 3, (n * 6) // 7]):
        for fill in (torch.zeros(2, n), torch.full((2, n), float("-inf")), base.clamp(max=1.0)):
            spikes = fill.clone()
            spikes[:, at] = torch.arange(len(at), 0, -1).float() + 7.0
            rows.append(spikes)
    for x in rows:
        for k in (n // 8, n // 4):
            _check(x.to(t), k)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 200000, 30000), (1, 1 << 20, 1 << 18), (3, 9 * 16384 + 1, 1000)])
def test_runs_of_ties_and_neighbours_that_go_together(shape, dtype):
    """Rows that are cut between elements of the sample, bins of many ties on a short stretch of the row, bins past what LDS holds."""
    m, n, k = shape
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    base = workloads.normal_rows(m, n, seed=n % 983)
    stairs = (torch.arange(n) // 3000).float().repeat(m, 1)
    lagged = torch.nn.functional.avg_pool1d(base.unsqueeze(1), 65, 1, 32).squeeze(1) * 8.0
    spikes = torch.zeros(m, n)
    spikes[:, 5] = 2.0
    spikes[:, (n * 7) // 9] = 1.0
    stripes = base.clone()
    stripes[:, (torch.arange(n) // 4096) % 2 == 0] = float("-inf")
    two = torch.full((m, n), 0.3)
    two[:, n // 2: n // 2 + k // 2] = 0.7
    for x in (torch.full((m, n), 0.3), stairs, -stairs, lagged, base.cumsum(1) / n ** 0.5, spikes, stripes, two, torch.relu(base - 1.5),
              torch.randint(0, 3, (m, n)).float(), torch.randint(0, 1000, (m, n)).float(), base + torch.linspace(0.0, 6.0, n)):
        _check(x.to(t).contiguous(), k, shift=n % 2)


def test_many_long_bf16_rows():
    _check(workloads.normal_rows(64, 1 << 21, seed=11, dtype="bf16"), 1 << 19)


def _check_pairs(x, k, b, k_b, assignment=None):
    vals, idx = atk.approx_topk(x.cuda(), k, b, k_b, assignment=assignment)
    torch.cuda.synchronize()
    ov, oi = oracle.approx_topk(workloads.as_numpy_bits(x), k, b, k_b, threads=8,
                                assignment=oracle.CONTIGUOUS if assignment == atk.ATK_CONTIGUOUS else oracle.INTERLEAVED)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(_bits(vals), ov.view(np.uint32) if ov.dtype == np.float32 else ov)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pairs(dtype):
    """Stage 2 over long lists of (value, index) pairs."""
    for (m, n, k, b, k_b) in [(2, 600000, 20000, 70001, 1), (1, 1 << 20, 40000, 1 << 16, 2)]:
        _check_pairs(workloads.normal_rows(m, n, seed=b, dtype=dtype), k, b, k_b)
        x = workloads.normal_rows(m, n, seed=b, dtype=dtype)
        x[:, : n // 4] = float("-inf")
        _check_pairs(x, k, b, k_b, assignment=atk.ATK_CONTIGUOUS)
        x[:, : n // 4] = 0.0
        _check_pairs(x, k, b, k_b, assignment=atk.ATK_CONTIGUOUS)
