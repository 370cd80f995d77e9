"""Scattered rows with buckets that the second cut cannot part: the bitonic network, at every row size.

One column met by more B rows than the kernel compares in a bucket: equal
columns share every bucket, so the row is sorted by the network.  The windows
are wider than the bit-window kernels take, so the rows can go nowhere else; the
statistics say that they did not.
"""
import os
import re

import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1801_03065_amd", "csrc",
                   "spg_bucket.hip")
K = 3_000_000


def _deep():
    return int(re.search(r"constexpr int BK_DEEP = (\d+);", open(SRC).read()).group(1))


def _product(f, na, hot, rows, seed, near=None):
    """Rows of f products: columns hot[j] = (column, B rows that hold it), the rest met once, spread or `near` one place."""
    rng = np.random.default_rng(seed)
    ci, lens = [], []
    for _ in range(rows):
        b = [[] for _ in range(na)]
        for c, times in hot:
            for r in rng.choice(na, times, replace=False):
                b[r].append(c)
        left = f - sum(t for _, t in hot) - 2
        pool = rng.choice(K - 200, 4 * f + 400, replace=False) + 100 if near is None else near + rng.permutation(4 * f + 400)
        rest = np.setdiff1d(pool, [c for c, _ in hot])
        for c in np.concatenate([[3, K - 3], rng.permutation(rest)[:left]]):  # both ends in every row: a wide window
            b[rng.integers(na)].append(int(c))
        for r in b:
            ci.append(np.unique(r).astype(np.int32))
            assert len(ci[-1]) == len(r)
            lens.append(len(r))
    n = rows * na
    A = synth.Csr(rows, n, np.arange(0, n + 1, na, dtype=np.int64), np.arange(n, dtype=np.int32), rng.standard_normal(n))
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    B = synth.Csr(n, K, rp, np.concatenate(ci), rng.standard_normal(int(rp[-1])))
    return A, B


@pytest.mark.parametrize("dtype,opts", [("f64", {}), ("f32", {}), ("f32", {"fp32_mode": 1}), ("f32", {"fp32_mode": 2})])
@pytest.mark.parametrize("f", [66, 100, 128, 129, 200, 256, 257, 400, 512, 513, 1000, 1024, 1025, 1500, 2048])
def test_equal_columns(f, dtype, opts):
    na = 40
    times = min(40, (f - 2) // 2)
    hot = [(1_234_567, times)] if f < 200 else [(1_234_567, times), (1_234_700, 30), (77, 26)]
    assert max(t for _, t in hot) > _deep()
    A, B = _product(f, na, hot, 14, f)
    if dtype == "f32":
        A, B = f32_inputs(A), f32_inputs(B)
    ref, S = oracle_ref(A, B)
    assert all(f <= 2 * n for n in np.diff(ref.row_ptr))
    got, h = run(A, B, dtype=dtype, **opts)
    st = h.stats()
    assert st["rows_scattered_numeric"] == 14 and st["rows_scattered_symbolic"] == 14
    assert st["rows_numeric"]["word_hash_wave"] == 14 and st["rows_symbolic"]["hash_wave"] == 14
    if dtype == "f64":
        check_f64(ref, S, got)
    else:  # at most 40 products an entry: gamma_40 and the rounded products, one rounding for the others
        check_f32(ref, S, got, rel=41 * 2.0**-24 * 1.01 if not opts else 6.1e-8)


@pytest.mark.parametrize("f", [90, 150, 300, 700, 1900])
def test_clustered_columns_beside_two_far_ones(f):
    """All columns but two in one bucket of the first cut; the second cut or the network orders them."""
    A, B = _product(f, 30, [(1_500_000, min(30, f // 4))] if f % 100 else [], 12, f, near=1_500_100)
    ref, S = oracle_ref(A, B)
    got, h = run(A, B)
    assert h.stats()["rows_scattered_numeric"] == 12
    check_f64(ref, S, got)
