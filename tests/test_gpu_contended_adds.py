"""FP32 sums in LDS under contention: many products of a row on few columns.

Values are small integers and every partial sum is below 2^24, so FP32 sums
are exact in any order and the GPU must give the oracle's values bit for bit,
whichever way an add took (compare-and-swap, or the atomic add after the
tries are spent).  The output widths put up to 64 lanes of a wavefront on one
address; the row sizes reach the team, wavefront and segment kernels.
"""
import numpy as np
import pytest

import oracle
import synth
from helpers import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("acc", [0, 1, 2, 3])
@pytest.mark.parametrize("per_a,per_b,k", [(60, 1, 1), (300, 1, 1), (64, 2, 2), (200, 3, 7), (40, 30, 33),
                                           (300, 40, 6000)])
def test_fp32_contended_sums_are_exact(per_a, per_b, k, acc):
    n = 400
    A = synth.random_csr(70, n, np.full(70, per_a), 1, "int")
    B = synth.random_csr(n, k, np.full(n, per_b), 2, "int")
    ref = oracle.spgemm(A, B)
    got, _ = run(A, B, dtype="f32", accumulator=acc, fp32_terms_max=0)
    assert np.array_equal(got[0], ref.row_ptr)
    assert np.array_equal(got[1], ref.col_idx)
    assert np.array_equal(got[2].astype(np.float64), ref.values)
