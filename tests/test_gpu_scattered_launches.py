"""Scattered rows: each launch of its own, launches joined, and rows whose columns repeat, against the oracle."""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu


def _product(sizes, na, k, seed, pick=None):
    """A row per size: na entries of A, B rows of its own with `size` columns in all (of `pick` where given)."""
    rng = np.random.default_rng(seed)
    sizes = np.asarray(sizes)
    m = len(sizes)
    lens = (sizes[:, None] * np.arange(1, na + 1) // na - sizes[:, None] * np.arange(na) // na).reshape(-1)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    A = synth.Csr(m, m * na, np.arange(0, m * na + 1, na, dtype=np.int64), np.arange(m * na, dtype=np.int32),
                  rng.standard_normal(m * na))
    if pick is None:  # distinct, increasing: a random start and steps of at least one
        step = max(1, k // int(lens.max()) - 1)
        pos = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
        ci = pos * step + rng.integers(0, step, int(rp[-1]))
    else:
        ci = np.concatenate([np.sort(rng.choice(pick, n, replace=False)) for n in lens])
    return A, synth.Csr(m * na, k, rp, ci.astype(np.int32), rng.standard_normal(int(rp[-1])))


@pytest.mark.parametrize("f", [99, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048])
def test_a_launch_of_its_own(f):
    """Too many rows to join the next launch (over 8 per CU of 256), with one larger row that has its own."""
    A, B = _product([f] * 2100 + [2 * f if f <= 1024 else f], 16, 2_000_000, f)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, B)
    check_f64(ref, S, got)


def test_joined_launches():
    """A few rows of every size class, in one launch."""
    A, B = _product([97, 128, 129, 250, 300, 512, 600, 1024, 1100, 2048] * 5, 24, 2_000_000, 3)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, B)
    check_f64(ref, S, got)


@pytest.mark.parametrize("f", [120, 480, 1000, 2040])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_many_repeats_of_few_columns(dtype, f):
    """Half of a row's products fall on two columns (each B row holds both), the rest are spread: deep buckets."""
    na = 60
    A, B = _product([2 * na] * 40, na, 3_000_000, f, np.array([77, 2_500_000]))
    C, D = _product([f - 60] * 40, na, 2_400_000, f + 1)
    # rows of B: the two popular columns, and f - 60 spread ones over the row's B rows
    rp = B.row_ptr + D.row_ptr
    ci = np.concatenate([np.sort(np.concatenate([B.col_idx[B.row_ptr[i]:B.row_ptr[i + 1]],
                                                 100 + D.col_idx[D.row_ptr[i]:D.row_ptr[i + 1]]]))
                         for i in range(B.nrows)])
    B = synth.Csr(B.nrows, 3_000_000, rp, ci.astype(np.int32), np.random.default_rng(f).standard_normal(len(ci)))
    if dtype == "f32":
        A, B = f32_inputs(A), f32_inputs(B)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, B, dtype=dtype)
    if dtype == "f64":
        check_f64(ref, S, got)
    else:  # at most 60 products an entry: gamma_60 with unit roundoff 2^-24, and the final rounding
        check_f32(ref, S, got, rel=61 * 2.0**-24 * 1.01)
