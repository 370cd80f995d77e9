"""Row statistics of an unsorted B: rows at the edges of the in-place counts (16
entries with one lane per row, 64 with 16 lanes), longer rows, rows wider than
the bitmap, mixed with sorted rows.  The compressed flop count must equal the
count of distinct column-set words by the oracle, and C the oracle's."""
import numpy as np
import pytest

import oracle
import synth
from helpers import check_f64, oracle_ref, run

pytestmark = pytest.mark.gpu


def _b(lens, k, seed, every=0):
    """Rows of the given lengths; every `every`-th is left sorted (0: none)."""
    B = synth.random_csr(lens.size, k, lens, seed)
    S = synth.shuffle_columns(B, seed + 1)
    ci = S.col_idx.copy()
    for i in range(lens.size):
        if every and i % every == 0:
            ci[B.row_ptr[i]:B.row_ptr[i + 1]] = B.col_idx[B.row_ptr[i]:B.row_ptr[i + 1]]
    return synth.Csr(S.nrows, S.ncols, S.row_ptr, ci, S.values)


@pytest.mark.parametrize("k", [300, 60_000])
@pytest.mark.parametrize("every", [0, 2])
@pytest.mark.parametrize("short", [True, False])  # average row length up to 8, and beyond
def test_word_counts_of_unsorted_rows(short, every, k):
    edge = np.array([0, 1, 2, 15, 16, 17, 18, 31, 32, 33, 63, 64, 65, 66, 128, 200])
    lens = np.concatenate([edge, edge, np.full(400 if short else 40, 4 if short else 30)])
    assert (lens.mean() <= 8) == short
    B = _b(lens, k, 3, every)
    A = synth.shuffle_columns(synth.random_csr(200, lens.size, np.full(200, 9), 5), 6)
    ref, S = oracle_ref(A, B)
    want = int(oracle.block_counts(B, 32)[A.col_idx].sum())
    for comp in (-1, 0, 1):
        got, h = run(A, B, compression=comp)
        check_f64(ref, S, got)
        assert h.stats()["flops_compressed"] == want


@pytest.mark.parametrize("per", [6, 40])
def test_rows_wider_than_the_bitmap(per):
    """Windows past 2^19 columns: compression is skipped, the product is the oracle's."""
    B = _b(np.full(300, per), (1 << 20) + 500, 8)
    A = synth.random_csr(100, 300, np.full(100, 12), 9)
    ref, S = oracle_ref(A, B)
    for comp in (-1, 1):
        got, h = run(A, B, compression=comp)
        check_f64(ref, S, got)
        assert h.stats()["compressed"] == 0
