"""Rows of many multiplications and few entries, on both sides of the workgroup rule, against the oracle."""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu


def _product(k, seed):
    """B: 300 rows of 64 columns; A's rows take 1 to 200 of them: 64 to 12800 multiplications, 4096 among them."""
    rng = np.random.default_rng(seed)
    B = synth.random_csr(300, k, np.full(300, 64), seed)
    counts = np.array([1, 2, 30, 63, 64, 65, 66, 100, 128, 129, 200] * 3)
    rp = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    ci = np.concatenate([np.sort(rng.choice(300, c, replace=False)) for c in counts]).astype(np.int32)
    return synth.Csr(len(counts), 300, rp, ci, rng.standard_normal(len(ci))), B


@pytest.mark.parametrize("k", [65, 500, 2048, 100_000])
@pytest.mark.parametrize("dtype,opts", [("f64", {}), ("f32", {}), ("f32", {"fp32_mode": 1}), ("f32", {"fp32_mode": 2})])
def test_long_rows(dtype, opts, k):
    A, B = _product(k, k)
    if dtype == "f32":
        A, B = f32_inputs(A), f32_inputs(B)
    ref, S = oracle_ref(A, B)
    got, h = run(A, B, dtype=dtype, **opts)
    if dtype == "f64":
        check_f64(ref, S, got)
        assert h.stats()["rows_symbolic"]["dense_wg"] >= 15  # more than 4096 multiplications
    else:  # at most 200 products an entry: gamma_200 for plain sums, one rounding and FP64's for the others
        check_f32(ref, S, got, rel=201 * 2.0**-24 * 1.01 if not opts else 6.1e-8)


def test_long_rows_of_unsorted_b():
    A, B = _product(2048, 7)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, synth.shuffle_columns(B, 1))
    check_f64(ref, S, got)
