"""A row of B that repeats columns (outside the contract, but summed all the same) longer than its window."""
import numpy as np
import pytest

import synth
from helpers import check_f64, oracle_ref, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("compression", [-1, 0])
def test_more_entries_than_window_columns(compression):
    cols = np.concatenate([np.arange(20_000), np.arange(80_000)]).astype(np.int32)
    rng = np.random.default_rng(1)
    B = synth.Csr(2, 90_000, np.array([0, cols.size, cols.size + 3], np.int64),
                  np.concatenate([cols, [5, 3, 70_000]]).astype(np.int32), rng.standard_normal(cols.size + 3))
    A = synth.Csr(3, 2, np.array([0, 2, 3, 4], np.int64), np.array([0, 1, 0, 1], np.int32), rng.standard_normal(4))
    ref, S = oracle_ref(A, B)
    assert np.array_equal(np.diff(ref.row_ptr), [80_000, 80_000, 3])
    got, _ = run(A, B, compression=compression)
    check_f64(ref, S, got)
