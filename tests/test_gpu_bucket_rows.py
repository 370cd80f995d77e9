"""Scattered rows in column buckets against the oracle.

The row sizes sit at the edges of the kernel's launches (128, 256, 512, 1024
and 2048 multiplications) and of its rule (64 A entries, two products per
entry, 2^20-column windows and beyond); columns are spread evenly, clustered
(one bucket holds most of the row: the sorting network), or repeated.
"""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, dev, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu


def _rows(products, na, k, seed, cols=None):
    """Rows of A with na entries each, whose B rows hold products[i] columns in all; B rows are not shared."""
    rng = np.random.default_rng(seed)
    lens = []
    for f in products:
        cuts = np.sort(rng.integers(0, f + 1, na - 1))
        lens.append(np.diff(np.concatenate([[0], cuts, [f]])))
    lens = np.concatenate(lens)
    m = len(products)
    A = synth.Csr(m, m * na, np.arange(0, m * na + 1, na, dtype=np.int64), np.arange(m * na, dtype=np.int32),
                  rng.standard_normal(m * na))
    if cols is None:
        B = synth.random_csr(m * na, k, np.minimum(lens, k), seed + 1)
    else:
        rp = np.concatenate([[0], np.cumsum(lens)])
        ci = np.concatenate([np.sort(rng.choice(cols, n, replace=False)) for n in lens]) if lens.sum() else lens
        B = synth.Csr(m * na, k, rp.astype(np.int64), ci.astype(np.int32), rng.standard_normal(int(rp[-1])))
    return A, B


EDGES = [65, 66, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1000, 1023, 1024, 1025, 1500, 2047, 2048, 2049]


@pytest.mark.parametrize("k", [70_000, 3_000_000])
@pytest.mark.parametrize("na", [3, 40, 64, 65])
def test_row_sizes_at_launch_edges(na, k):
    A, B = _rows(EDGES * 3, na, k, na + k)
    ref, S = oracle_ref(A, B)
    got, h = run(A, B)
    check_f64(ref, S, got)
    if na <= 64 and k > 1 << 20:
        assert h.stats()["rows_numeric"]["word_hash_wave"] >= 3 * (len(EDGES) - 1)
    got, _ = run(A, synth.shuffle_columns(B, 5))
    check_f64(ref, S, got)


@pytest.mark.parametrize("dtype,opts", [("f64", {}), ("f32", {}), ("f32", {"fp32_mode": 1}), ("f32", {"fp32_mode": 2})])
def test_repeated_columns(dtype, opts):
    """Up to two products per entry on average, some columns met by most B rows."""
    cols = np.concatenate([np.arange(8) * 7, np.arange(100, 2_000_000, 5003)])
    A, B = _rows([100, 200, 250, 400, 500, 700, 800, 1300] * 4, 20, 2_000_000, 9, cols)
    if dtype == "f32":
        A, B = f32_inputs(A), f32_inputs(B)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, B, dtype=dtype, **opts)
    if dtype == "f64":
        check_f64(ref, S, got)
    else:  # at most 20 products an entry: gamma_20 for plain sums, one rounding for the others
        check_f32(ref, S, got, rel=1.3e-6 if not opts else 6.1e-8)


@pytest.mark.parametrize("f", [90, 300, 1024, 1900])
def test_clustered_columns_take_the_network(f):
    """All but two columns of a row in one bucket of its window."""
    cols = np.concatenate([np.arange(1_000_000, 1_000_000 + 1800), [5, 2_999_000]])
    A, B = _rows([f] * 12, 30, 3_000_000, f, cols)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, B)
    check_f64(ref, S, got)


def test_panels_and_values_on_bucket_rows():
    import torch

    import paper_1801_03065_amd as spg

    A, B = _rows(EDGES * 2, 30, 2_000_000, 77)
    h = spg.Handle()
    dA, dB = dev(A), dev(B)
    rp, nnz = spg.spgemm_symbolic(h, dA, dB)
    C = spg.spgemm_numeric(h, dA, dB, rp, nnz)
    rph = rp.cpu().numpy().astype(np.int64)
    for rb, re_ in ((0, 7), (7, 8), (3, A.nrows)):
        n = int(rph[re_] - rph[rb])
        pc = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        pv = torch.zeros(n, dtype=torch.float64, device="cuda")
        spg.spgemm_numeric_rows(h, dA, dB, rb, re_, pc, pv)
        assert torch.equal(pc, C.col_idx[rph[rb]:rph[re_]]) and torch.equal(pv, C.values[rph[rb]:rph[re_]])
    A2 = synth.revalue(A, 3)
    d2 = dA.with_values(torch.as_tensor(A2.values, device="cuda"))
    spg.spgemm_numeric_values(h, d2, dB, C)
    h.check_errors()
    ref, S = oracle_ref(A2, B)
    check_f64(ref, S, (rph, C.col_idx.cpu().numpy(), C.values.cpu().numpy()))


def test_structure_changed_behind_the_plan_is_reported():
    import torch

    import paper_1801_03065_amd as spg

    A, B = _rows([300] * 6, 30, 2_000_000, 5)
    h = spg.Handle()
    dA, dB = dev(A), dev(B)
    rp, nnz = spg.spgemm_symbolic(h, dA, dB)
    dB.col_idx[0:2] = dB.col_idx[1].clone()  # one column twice in a row of B: a smaller row of C
    dB.col_idx.copy_(torch.zeros_like(dB.col_idx))
    spg.spgemm_numeric(h, dA, dB, rp, nnz)
    with pytest.raises(spg.SpgemmError):
        h.check_errors()
