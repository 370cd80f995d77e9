"""Heavy rows: the stored bit windows and the symbolic window kernel at its edges.

Windows of one and several aligned groups of 4096 words and beyond 8192 words
(the 1024-lane symbolic launch), rows with more multiplications than window
words (window kept) and fewer (rebuilt), A rows of one and several chunks,
popular columns that most B rows share, compressed and raw B.
"""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, dev, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu


def _pair(k, la, lb, seed, hot=0, runs=1):
    rng = np.random.default_rng(seed)
    n = 1500
    A = synth.random_csr(8, n, np.resize(la, 8), seed)
    B0 = synth.random_csr(n, k // runs - 1, rng.integers(lb // 2, lb + 1, n), seed + 1)
    rows = [B0.col_idx[B0.row_ptr[i]:B0.row_ptr[i + 1]].astype(np.int64) * runs for i in range(n)]
    extra = rng.integers(0, k, hot)
    rows = [np.unique(np.concatenate([(r[:, None] + np.arange(runs)).reshape(-1), extra])) for r in rows]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    ci = np.concatenate(rows).astype(np.int32)
    return A, synth.Csr(n, k, rp, ci, rng.standard_normal(ci.size))


CASES = [  # columns, A entries, B entries, popular columns, columns per run
    (90_000, (60, 300, 700, 1300), 90, 0, 1),
    (131_072, (60, 511, 512, 513), 120, 12, 1),
    (140_000, (100, 1025), 100, 0, 16),       # two groups, compressed B
    (262_144 + 33, (80, 600), 100, 5, 1),     # past 8192 words
    (1_000_000, (50, 900), 110, 8, 1),        # fewer multiplications than words in the short rows
    (1_048_576, (1200,), 200, 0, 1),
]


@pytest.mark.parametrize("compression", [-1, 0, 1])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_heavy_windows(case, compression):
    k, la, lb, hot, runs = CASES[case]
    A, B = _pair(k, la, lb, case + 10, hot, runs)
    ref, S = oracle_ref(A, B)
    got, h = run(A, B, compression=compression)
    check_f64(ref, S, got)
    assert h.stats()["rows_numeric"]["dense_wg"] > 0
    A32, B32 = f32_inputs(A), f32_inputs(B)
    ref32, S32 = oracle_ref(A32, B32)
    got, _ = run(A, B, dtype="f32", compression=compression)
    check_f32(ref32, S32, got)


def test_one_plan_reused_then_replaced():
    """New values on a plan with kept windows, then another structure on the same handle, then the first again."""
    import torch

    import paper_1801_03065_amd as spg

    h = spg.Handle()
    for case in (0, 4, 1, 0):
        k, la, lb, hot, runs = CASES[case]
        A, B = _pair(k, la, lb, case + 40, hot, runs)
        dA, dB = dev(A), dev(B)
        rp, nnz = spg.spgemm_symbolic(h, dA, dB)
        for seed in (1, 2):
            A2 = synth.revalue(A, seed)
            d2 = dA.with_values(torch.as_tensor(A2.values, device="cuda"))
            C = spg.spgemm_numeric(h, d2, dB, rp, nnz)
            h.check_errors()
            ref, S = oracle_ref(A2, B)
            check_f64(ref, S, (rp.cpu().numpy().astype(np.int64), C.col_idx.cpu().numpy(), C.values.cpu().numpy()))
