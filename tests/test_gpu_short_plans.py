"""Plans whose rows are all short rows (their symbolic row lists serve the
numeric phase): error checks between calls, panels, values only, autotuning,
forced compression, rows without products, a separate FP64 row set, and the
same handle before and after on products of other kinds."""
import numpy as np
import pytest

import oracle
import synth
from helpers import check_f32, check_f64, dev, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu


def _got(rp, C):
    return rp.cpu().numpy().astype(np.int64), C.col_idx.cpu().numpy(), C.values.cpu().numpy()


def _short(seed=1):
    A = synth.random_csr(3000, 2500, np.random.default_rng(seed).integers(0, 6, 3000), seed)
    B = synth.random_csr(2500, 1800, np.random.default_rng(seed + 1).integers(0, 9, 2500), seed + 1)
    return A, B


@pytest.mark.parametrize("opts", [{}, {"autotune": 1}, {"compression": 1}, {"verify_structure": 1}])
@pytest.mark.parametrize("rp", ["i32", "i64"])
def test_all_short_plan(opts, rp):
    import torch

    import paper_1801_03065_amd as spg

    A, B = _short()
    h = spg.Handle(**opts)
    dA, dB = dev(A, rp=rp), dev(B, rp=rp)
    ref, S = oracle_ref(A, B)
    rpt, nnz = spg.spgemm_symbolic(h, dA, dB, dA.row_ptr.dtype)
    st = h.stats()
    assert nnz == ref.nnz and st["rows_symbolic"]["short_rows"] + st["rows_symbolic"]["empty"] == A.nrows
    assert st["nnz_b_compressed"] == (int(oracle.block_counts(B, 32).sum()) if opts.get("compression") else 0)
    for _ in range(3):
        C = spg.spgemm_numeric(h, dA, dB, rpt, nnz)
        h.check_errors()
        check_f64(ref, S, _got(rpt, C))
    A2 = synth.revalue(A, 7)
    d2 = dA.with_values(torch.as_tensor(A2.values, device="cuda"))
    ref2, S2 = oracle_ref(A2, B)
    for _ in range(2):
        spg.spgemm_numeric_values(h, d2, dB, C)
        h.check_errors()
        check_f64(ref2, S2, _got(rpt, C))
    for rb, re_ in ((0, 1), (700, 1900), (0, A.nrows)):
        n = int(ref.row_ptr[re_] - ref.row_ptr[rb])
        pc = torch.full((max(n, 1),), -7, dtype=torch.int32, device="cuda")
        pv = torch.zeros(max(n, 1), dtype=torch.float64, device="cuda")
        spg.spgemm_numeric_rows(h, d2, dB, rb, re_, pc, pv)
        h.check_errors()
        assert np.array_equal(pc.cpu().numpy()[:n], ref2.col_idx[ref2.row_ptr[rb]:ref2.row_ptr[re_]])
        assert np.allclose(pv.cpu().numpy()[:n], ref2.values[ref2.row_ptr[rb]:ref2.row_ptr[re_]], rtol=0, atol=1e-12)


def test_handle_alternates_between_plans():
    import paper_1801_03065_amd as spg

    h = spg.Handle()
    big = synth.stencil27(9)
    wide = synth.random_csr(500, 3000, np.random.default_rng(4).integers(0, 40, 500), 4)
    cols = synth.random_csr(3000, 400_000, np.random.default_rng(5).integers(0, 30, 3000), 5)
    for A, B in (_short(), (big, big), _short(3), (wide, cols), _short(5), _short(5)):
        dA, dB = dev(A), dev(B)
        rp, nnz = spg.spgemm_symbolic(h, dA, dB)
        C = spg.spgemm_numeric(h, dA, dB, rp, nnz)
        h.check_errors()
        C = spg.spgemm_numeric(h, dA, dB, rp, nnz)
        ref, S = oracle_ref(A, B)
        check_f64(ref, S, _got(rp, C))


def test_short_rows_past_the_fp32_term_limit():
    """Rows of 300 A entries that meet mostly empty B rows: short rows with a separate FP64 row set."""
    lens = np.where(np.arange(400) % 5 == 0, 300, 4)
    A = synth.random_csr(400, 4000, lens, 1)
    B = synth.random_csr(4000, 500, (np.arange(4000) % 8 == 0).astype(np.int64), 2)
    A32, B32 = f32_inputs(A), f32_inputs(B)
    ref, S = oracle_ref(A32, B32)
    got, h = run(A, B, dtype="f32")
    check_f32(ref, S, got)
    assert h.stats()["fp64_rows"] == 80


@pytest.mark.parametrize("m,n,k", [(0, 5, 5), (5, 0, 5), (5, 5, 0), (1, 1, 1), (2049, 3, 3)])
def test_degenerate_shapes(m, n, k):
    A = synth.random_csr(m, n, np.minimum(np.full(m, 2), n), 1)
    B = synth.random_csr(n, k, np.minimum(np.full(n, 2), k), 2)
    ref, S = oracle_ref(A, B)
    for crp in ("i32", "i64"):
        got, h = run(A, B, crp=crp)
        check_f64(ref, S, got)
