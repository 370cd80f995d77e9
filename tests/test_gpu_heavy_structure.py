"""Heavy rows whose bit windows the plan keeps, met by other products than the plan's.

B's columns are changed behind the plan (same row lengths, rows sorted): a heavy
row that loses or gains a column differs in size from the plan and is reported;
a row of the same size is the product of what B holds now.  Stored zeros are
products like others.  Rows of one and several chunks of A entries, of one and
several segments.
"""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, dev, f32_inputs, oracle_ref

pytestmark = pytest.mark.gpu

# A entries per heavy row, columns, entries per row of B (multiplications above both 4096 and the window's words)
CASES = [(60, 90_000, 90), (700, 90_000, 90), (60, 60_000, 70), (400, 1_000_000, 100), (600, 3_000, 20)]


def _pair(na, k, lb, seed=3, rows=5):
    """Every row of C has B rows of its own."""
    n = na * rows
    A = synth.Csr(rows, n, np.arange(0, n + 1, na, dtype=np.int64), np.arange(n, dtype=np.int32),
                  np.random.default_rng(seed).standard_normal(n))
    B = synth.random_csr(n, k, np.full(n, lb), seed + 1)
    return A, synth.Csr(n, k + 400, B.row_ptr, B.col_idx, B.values)  # the last 400 columns are empty


def _changed(B, na, row, how):
    """B with one column of one of the row's B rows replaced; the C row loses or gains a column, or swaps one for its
    neighbour (same word)."""
    ci = B.col_idx.copy()
    lo, hi = B.row_ptr[row * na], B.row_ptr[(row + 1) * na]
    cols, cnt = np.unique(ci[lo:hi], return_counts=True)
    once, often = cols[cnt == 1], cols[cnt > 1]
    if how == "loses":
        pairs = [(c, d) for c in once[:50] for d in (cols[:50] if cols[0] != c else cols[1:50])]
    elif how == "gains beyond":
        pairs = [(c, k) for c in often[:50] for k in (cols[-1] + 300,)]
    elif how == "gains":
        pairs = [(c, d) for c in often[:50] for d in np.setdiff1d(np.arange(cols[0], cols[-1]), cols)[:50]]
    else:
        pairs = [(c, c ^ 1) for c in once if cols[0] < c < cols[-1] and (c ^ 1) not in cols]
    for c, d in pairs:
        at = lo + int(np.nonzero(ci[lo:hi] == c)[0][0])
        j = int(np.searchsorted(B.row_ptr, at, side="right")) - 1
        b, e = B.row_ptr[j], B.row_ptr[j + 1]
        if d in ci[b:e]:
            continue
        ci[at] = d
        ci[b:e] = np.sort(ci[b:e])
        return synth.Csr(B.nrows, B.ncols, B.row_ptr, ci, B.values)
    return None


def _plan(A, B, dtype, **opts):
    import paper_1801_03065_amd as spg

    h = spg.Handle(**opts)
    dA, dB = dev(A, dtype), dev(B, dtype)
    rp, nnz = spg.spgemm_symbolic(h, dA, dB)
    assert h.stats()["rows_numeric"]["dense_wg"] == A.nrows
    return h, dA, dB, rp, nnz


@pytest.mark.parametrize("dtype,opts", [("f64", {}), ("f32", {"fp32_terms_max": 0}), ("f32", {})])
@pytest.mark.parametrize("how", ["loses", "gains", "gains beyond", "swaps"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_changed_structure_of_heavy_rows(case, how, dtype, opts):
    import torch

    import paper_1801_03065_amd as spg

    na, k, lb = CASES[case]
    A, B = _pair(na, k, lb)
    B2 = _changed(B, na, 2, how)
    if B2 is None:
        pytest.fail("no such change in this case")
    h, dA, dB, rp, nnz = _plan(A, B, dtype, **opts)
    dB.col_idx.copy_(torch.as_tensor(B2.col_idx, device="cuda"))
    C = spg.spgemm_numeric(h, dA, dB, rp, nnz)
    if dtype == "f32":
        A, B2 = f32_inputs(A), f32_inputs(B2)
    ref, S = oracle_ref(A, B2)
    same = np.array_equal(np.asarray(ref.row_ptr), rp.cpu().numpy())
    assert same == (how == "swaps")
    if not same:
        with pytest.raises(spg.SpgemmError) as e:
            h.check_errors()
        assert e.value.status == spg.SPG_ERR_STRUCTURE_MISMATCH
        # the other rows are the plan's
        r = rp.cpu().numpy()
        keep = np.concatenate([np.arange(r[i], r[i + 1]) for i in (0, 1, 3, 4)])
        ref, S = oracle_ref(A, f32_inputs(B) if dtype == "f32" else B)
        err = np.abs(C.values.cpu().numpy()[keep].astype(np.float64) - ref.values[keep])
        assert np.array_equal(C.col_idx.cpu().numpy()[keep], ref.col_idx[keep])
        assert np.all(err <= (1e-12 if dtype == "f64" else 4.2e-5) * S[keep])
        return
    h.check_errors()
    got = (rp.cpu().numpy().astype(np.int64), C.col_idx.cpu().numpy(), C.values.cpu().numpy())
    if dtype == "f64":
        check_f64(ref, S, got)
    else:  # plain FP32 sums of at most na products (gamma_700 = 4.2e-5), FP64 ones beyond the term limit
        check_f32(ref, S, got, rel=4.2e-5)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_stored_zeros_of_heavy_rows(case, dtype):
    """Entries whose products are all zero, and a changed column among them."""
    import torch

    import paper_1801_03065_amd as spg

    na, k, lb = CASES[case]
    A, B = _pair(na, k, lb, seed=9)
    A.values[::2] = 0.0
    h, dA, dB, rp, nnz = _plan(A, B, dtype)
    C = spg.spgemm_numeric(h, dA, dB, rp, nnz)
    h.check_errors()
    ref, S = oracle_ref(f32_inputs(A), f32_inputs(B)) if dtype == "f32" else oracle_ref(A, B)
    got = (rp.cpu().numpy().astype(np.int64), C.col_idx.cpu().numpy(), C.values.cpu().numpy())
    (check_f64 if dtype == "f64" else check_f32)(ref, S, got)
    zero = got[2] == 0
    assert zero.any() and not np.signbit(got[2][zero]).any()  # sums start from 0.0
    # sums that cancel: exact in any order
    A1, B1 = A.with_values(np.sign(A.values) + (A.values == 0)), B.with_values(np.sign(B.values))
    d1, e1 = dA.with_values(torch.as_tensor(A1.values).to(dA.values)), dB.with_values(torch.as_tensor(B1.values).to(dB.values))
    C1 = spg.spgemm_numeric(h, d1, e1, rp, nnz)
    h.check_errors()
    assert np.array_equal(C1.values.cpu().numpy(), oracle_ref(A1, B1)[0].values.astype(got[2].dtype))
    B2 = _changed(B, na, 1, "loses")
    dB.col_idx.copy_(torch.as_tensor(B2.col_idx, device="cuda"))
    spg.spgemm_numeric(h, dA, dB, rp, nnz, out=C)
    with pytest.raises(spg.SpgemmError):
        h.check_errors()
