"""Rows of A and B at the analysis' long-row limit (256 entries) and far beyond it, against the oracle."""
import numpy as np
import pytest

import synth
from helpers import check_f64, oracle_ref, run

pytestmark = pytest.mark.gpu

LENS = [255, 256, 257, 319, 320, 321, 511, 512, 513, 1000, 1025, 3000, 7777]


@pytest.mark.parametrize("compression", [-1, 0, 1])
@pytest.mark.parametrize("k", [8_000, 400_000])
@pytest.mark.parametrize("short", [0, 6000])
def test_long_rows_of_b(short, k, compression):
    """Dense runs and spread columns; with many empty rows the one-lane-per-row kernels run."""
    rng = np.random.default_rng(k + short)
    rows = []
    for n in LENS:
        rows.append(np.sort(rng.choice(k, n, replace=False)))
        rows.append(np.arange(n) + 13)                        # whole words, starting inside one
        rows.append(np.sort(rng.choice(min(k, n + 40), n, replace=False)))  # nearly whole words
    rows += [np.sort(rng.choice(k, c, replace=False)) for c in rng.integers(0, 4, short)]
    order = rng.permutation(len(rows))
    rows = [rows[i] for i in order]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    B = synth.Csr(len(rows), k, rp, np.concatenate(rows).astype(np.int32), rng.standard_normal(int(rp[-1])))
    A = synth.random_csr(200, len(rows), rng.integers(0, 6, 200), 5)
    eye = np.arange(len(rows))
    A = synth.Csr(200 + len(rows), len(rows), np.concatenate([A.row_ptr, A.row_ptr[-1] + 1 + eye]),
                  np.concatenate([A.col_idx, eye]).astype(np.int32), rng.standard_normal(A.nnz + len(rows)))
    ref, S = oracle_ref(A, B)
    got, h = run(A, B, compression=compression)
    check_f64(ref, S, got)
    st = h.stats()
    lens = np.diff(rp)
    words = np.array([len(np.unique(r >> 5)) for r in rows])
    assert st["flops"] == lens[A.col_idx].sum() and st["flops_compressed"] == words[A.col_idx].sum()
    got, _ = run(A, synth.shuffle_columns(B, 3), compression=compression)
    check_f64(ref, S, got)


def test_long_rows_of_a():
    rng = np.random.default_rng(1)
    n = 9000
    B = synth.random_csr(n, 5000, rng.integers(0, 5, n), 2)
    rows = [np.sort(rng.choice(n, c, replace=False)) for c in LENS + [0, 1, 8000] + [3] * 50]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    A = synth.Csr(len(rows), n, rp, np.concatenate(rows).astype(np.int32), rng.standard_normal(int(rp[-1])))
    ref, S = oracle_ref(A, B)
    got, h = run(A, B)
    check_f64(ref, S, got)
    f = np.array([np.diff(B.row_ptr)[r].sum() for r in rows])
    assert h.stats()["flops"] == f.sum() and h.stats()["max_row_flops"] == f.max()


def test_bad_columns_in_long_rows_are_reported():
    import paper_1801_03065_amd as spg

    B = synth.random_csr(4, 5000, np.array([3, 2000, 5, 300]), 2)
    A = synth.random_csr(4, 4, np.full(4, 2), 3)
    ci = B.col_idx.copy()
    ci[1500] = 5000
    with pytest.raises(spg.SpgemmError):
        run(A, synth.Csr(4, 5000, B.row_ptr, ci, B.values))
    B = synth.random_csr(1000, 100, np.full(1000, 2), 2)
    A = synth.random_csr(2, 1000, np.array([600, 1]), 3)
    ci = A.col_idx.copy()
    ci[500] = -1
    with pytest.raises(spg.SpgemmError):
        run(synth.Csr(2, 1000, A.row_ptr, ci, A.values), B)
