"""Stored-structure rows in chunks of consecutive rows (B of 2^24 entries and more, FP64) and one by one, for every
number of lanes per row of B."""
import os
import re

import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1801_03065_amd", "csrc",
                   "spg_plan.hip")


@pytest.mark.parametrize("lb", [3, 6, 12, 24, 48, 100])
@pytest.mark.parametrize("side", [0, 1])
def test_chunks(lb, side):
    """B: bands of lb columns, 2^24 entries or a row less; A: 27 neighbouring rows of it, 1001 and 5 rows."""
    e = int(re.search(r"PL_CH_NNZ = int64_t\(1\) << (\d+);", open(SRC).read()).group(1))
    n = -(-(1 << e) // lb) if side else ((1 << e) - 1) // lb
    rng = np.random.default_rng(lb)
    cols = (np.arange(n, dtype=np.int32)[:, None] + np.arange(lb, dtype=np.int32)).reshape(-1)
    B = synth.Csr(n, n + lb, np.arange(0, n * lb + 1, lb, dtype=np.int64), cols, rng.standard_normal(n * lb))
    assert (B.nnz >= 1 << e) == bool(side)
    for m in (1001, 5):
        start = np.sort(rng.choice(n - 27, m, replace=False))
        A = synth.Csr(m, n, np.arange(0, 27 * m + 1, 27, dtype=np.int64),
                      (start[:, None] + np.arange(27)).reshape(-1).astype(np.int32), rng.standard_normal(27 * m))
        ref, S = oracle_ref(A, B)
        got, h = run(A, B)
        assert h.stats()["rows_numeric"]["planned_wave"] == m
        check_f64(ref, S, got)
        if side:
            ref, S = oracle_ref(f32_inputs(A), f32_inputs(B))
            got, _ = run(A, B, dtype="f32")
            check_f32(ref, S, got)
