"""The bins of exact_topk's row kernels, compiled for the host: a larger composite never lies in a lower bin, keys beyond the
upper end of the range among them, and edge() lies at or below everything in its bin."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2412_04358_amd", "csrc")

_SHIM = """
#include "atk_row_bins.h"
template <int ELT>
static void run(uint32_t lo, uint32_t hi, int idx_bits, int n_bins, const uint32_t *key, const uint32_t *idx, int64_t n, uint32_t *bin,
                uint32_t *edge) {
    atk::RowBins b;
    b.set<ELT>(lo, hi, idx_bits, n_bins);
    for (int64_t i = 0; i < n; ++i) {
        bin[i] = b.bin<ELT, true>(key[i], 0x7fffffffu - idx[i]);
        if (key[i] <= hi && b.bin<ELT>(key[i], 0x7fffffffu - idx[i]) != bin[i]) bin[i] = 0xffffffffu;
        edge[i] = b.edge<ELT>(bin[i]);
    }
}
extern "C" void row_bins(int bf16, uint32_t lo, uint32_t hi, int idx_bits, int n_bins, const uint32_t *key, const uint32_t *idx,
                         int64_t n, uint32_t *bin, uint32_t *edge) {
    if (bf16)
        run<ATK_BF16>(lo, hi, idx_bits, n_bins, key, idx, n, bin, edge);
    else
        run<ATK_F32>(lo, hi, idx_bits, n_bins, key, idx, n, bin, edge);
}
"""


@pytest.fixture(scope="module")
def row_bins(tmp_path_factory):
    where = tmp_path_factory.mktemp("row_bins")
    src, lib = where / "shim.cpp", where / "shim.so"
    src.write_text(_SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", _CSRC, "-o", str(lib), str(src)])
    f = ctypes.CDLL(str(lib)).row_bins
    p = ctypes.c_void_p
    f.argtypes = [ctypes.c_int, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int, ctypes.c_int, p, p, ctypes.c_int64, p, p]

    def call(bf16, lo, hi, idx_bits, n_bins, key, idx):
        key, idx = np.ascontiguousarray(key, dtype=np.uint32), np.ascontiguousarray(idx, dtype=np.uint32)
        bins, edges = np.empty_like(key), np.empty_like(key)
        f(bf16, lo, hi, idx_bits, n_bins, key.ctypes.data, idx.ctypes.data, len(key), bins.ctypes.data, edges.ctypes.data)
        return bins, edges

    return call


_TOP = 0xff800000  # the key of +inf


def _bf16_keys():
    """The order keys of all bf16 numbers, smallest first."""
    bits = np.arange(1 << 16, dtype=np.uint64) << 16
    bits = bits[((bits & 0x7fffffff) <= 0x7f800000) & (bits != 0x80000000)]
    return np.sort(np.where(bits >> 31, bits ^ 0xffffffff, bits ^ 0x80000000))


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("idx_bits", [1, 11, 17, 20, 21, 31])
@pytest.mark.parametrize("span", [0, 1, 300, 1 << 22, 0x7f000000])
@pytest.mark.parametrize("lo", [0x007fffff, 0x7f000000, 0x80000000, 0xbf800000, 0xbf801234])
def test_bins_keep_the_order(row_bins, bf16, idx_bits, span, lo):
    rng = np.random.default_rng(span + idx_bits)
    if bf16:  # (span counts keys; the lower end may also be a key without its low bits)
        keys = _bf16_keys()
        keys = keys[np.searchsorted(keys, lo):]
        at = min(span, len(keys) - 1)
        hi, inside, above = int(keys[at]), keys[rng.integers(0, at + 1, 4000)], keys[rng.integers(at, len(keys), 2000)]
        just_above = keys[np.minimum(at + rng.integers(0, 4, 500), len(keys) - 1)]
        lo = min(lo, int(keys[0]))
    else:
        hi = min(lo + span, _TOP)
        inside, above = rng.integers(lo, hi + 1, 4000), rng.integers(hi, _TOP + 1, 2000)
        just_above = np.minimum(hi + rng.integers(0, 4, 500), _TOP)
    key = np.concatenate([inside, above, just_above, np.full(2000, inside.min()), np.full(2000, hi)]).astype(np.int64)
    idx = rng.integers(0, 1 << idx_bits, len(key))
    order = np.lexsort((-idx, key))  # smallest composite first
    key, idx = key[order], idx[order]
    for n_bins in (256, 4096, 8192):
        bins, edges = row_bins(bf16, lo, hi, idx_bits, n_bins, key, idx)
        assert bins.max() < n_bins
        assert (np.diff(bins.astype(np.int64)) >= 0).all()
        within = key <= hi
        assert (edges[within] <= key[within]).all()


def test_keys_above_the_range_go_to_the_last_bin(row_bins):
    """A sample's largest key as the upper end, larger elements anywhere in the row: found wrong for -inf / 3.5 and 0.5 / 3.5."""
    for bf16, lo, hi, high in [(0, 0x007fffff, 0x007fffff, 0xc0600000), (1, 0x007fffff, 0xbf000000, 0xc0600000)]:
        bins, _ = row_bins(bf16, lo, hi, 20, 4096, [hi, high, high], [5, 5, 900000])
        assert list(bins) == [4095, 4095, 4095]
