"""Infinities and NaN reach exactly the entries their products belong to, in every numeric kernel."""
import numpy as np
import pytest

import oracle
import synth
from helpers import dev, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu


def _spoil(M, seed, share):
    """Infinities of both signs, NaN, zeros, and magnitudes whose products an FP32 still holds among the values."""
    rng = np.random.default_rng(seed)
    v = M.values.copy()
    at = rng.random(v.size) < share
    v[at] = rng.choice([np.inf, -np.inf, np.nan, 1e18, -1e18, 1e-18, 0.0, -0.0], int(at.sum()))
    return M.with_values(v)


def _same(want, S, got, rel):
    got = got.astype(np.float64)
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(want), np.isnan(got))
    assert np.array_equal(want[~fin & ~np.isnan(want)], got[~fin & ~np.isnan(want)])
    assert np.all(np.abs(got[fin] - want[fin]) <= rel * S[fin])


def _every_eighth(n, k, lb, seed):
    """More than 64 touched words a row and over two products an entry."""
    B = synth.random_csr(n, k, np.full(n, lb), seed)
    return synth.Csr(n, 8 * k, B.row_ptr, 8 * B.col_idx, B.values)


PAIRS = {  # kind of the rows: operands
    "short_rows": lambda: (synth.random_csr(4000, 3000, np.full(4000, 6), 1), synth.random_csr(3000, 9000, np.full(3000, 8), 2)),
    "column buckets": lambda: (synth.random_csr(300, 3000, np.full(300, 40), 3), synth.random_csr(3000, 2_500_000, np.full(3000, 20), 4)),
    "planned_wave": lambda: (synth.stencil27(12), synth.stencil27(12)),
    "word_hash_wave": lambda: (synth.random_csr(200, 300, np.full(200, 60), 5), _every_eighth(300, 1100, 40, 6)),
    "dense_wg": lambda: (synth.random_csr(12, 2000, np.resize([70, 700], 12), 7), synth.random_csr(2000, 90_000, np.full(2000, 90), 8)),
}


@pytest.mark.parametrize("dtype,opts", [("f64", {}), ("f32", {}), ("f32", {"fp32_mode": 2}), ("f64", {"accumulator": 1}),
                                        ("f64", {"accumulator": 2}), ("f32", {"accumulator": 1}), ("f32", {"accumulator": 2}),
                                        ("f64", {"accumulator": 3})])
@pytest.mark.parametrize("kind", list(PAIRS))
def test_product(kind, dtype, opts):
    A, B = PAIRS[kind]()
    A, B = _spoil(A, 1, 2e-3), _spoil(B, 2, 2e-3)
    if dtype == "f32":
        A, B = f32_inputs(A), f32_inputs(B)
    with np.errstate(invalid="ignore"):
        ref, S = oracle_ref(A, B)
    got, h = run(A, B, dtype=dtype, **opts)
    if not opts.get("accumulator"):
        st = h.stats()
        n = st["rows_scattered_numeric"] if kind == "column buckets" else st["rows_numeric"][kind]
        assert n > 0.9 * A.nrows
    assert np.array_equal(got[0], ref.row_ptr) and np.array_equal(got[1], ref.col_idx)
    _same(ref.values, S, got[2], 1e-12 if dtype == "f64" else 1e-5)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("kind", list(PAIRS))
def test_new_values_and_backward(kind, dtype):
    import torch

    import paper_1801_03065_amd as spg

    A, B = PAIRS[kind]()
    h, dA, dB = spg.Handle(), dev(A, dtype), dev(B, dtype)
    rp, nnz = spg.spgemm_symbolic(h, dA, dB)
    C = spg.spgemm_numeric(h, dA, dB, rp, nnz)
    A, B = _spoil(A, 3, 2e-3), _spoil(B, 4, 2e-3)
    if dtype == "f32":
        A, B = f32_inputs(A), f32_inputs(B)
    d2, e2 = (d.with_values(torch.as_tensor(M.values).to(d.values)) for d, M in ((dA, A), (dB, B)))
    spg.spgemm_numeric_values(h, d2, e2, C)
    h.check_errors()
    with np.errstate(invalid="ignore"):
        ref, S = oracle_ref(A, B)
        _same(ref.values, S, C.values.cpu().numpy(), 1e-12 if dtype == "f64" else 1e-5)
        # backward with a gradient of its own
        G = _spoil(ref.with_values(np.random.default_rng(5).standard_normal(ref.nnz)), 6, 1e-3)
        if dtype == "f32":
            G = f32_inputs(G)
        wa, wb = oracle.grad(A, B, ref, G.values)
        fin = lambda M: M.with_values(np.where(np.isfinite(M.values), np.abs(M.values), 0.0))
        sa, sb = oracle.grad(fin(A), fin(B), ref, fin(G).values)
    da, db = spg.spgemm_backward(h, d2, e2, C.with_values(torch.as_tensor(G.values).to(C.values)))
    h.check_errors()
    _same(wa, sa, da.cpu().numpy(), 1e-12 if dtype == "f64" else 1e-5)
    _same(wb, sb, db.cpu().numpy(), 1e-12 if dtype == "f64" else 1e-5)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_masked(dtype):
    import paper_1801_03065_amd as spg

    A = _spoil(synth.random_csr(60, 500, np.resize([5, 40, 300], 60), 1), 2, 5e-3)
    B = _spoil(synth.random_csr(500, 6000, np.full(500, 60), 3), 4, 5e-3)
    M = synth.random_csr(60, 6000, np.resize([100, 256, 900, 3000], 60), 5)
    if dtype == "f32":
        A, B = f32_inputs(A), f32_inputs(B)
    with np.errstate(invalid="ignore"):
        want, S = oracle.masked(A, B, M, with_abs=True)
    got = spg.spgemm_masked(spg.Handle(), dev(A, dtype), dev(B, dtype), dev(M, dtype)).cpu().numpy()
    _same(want, S, got, 1e-12 if dtype == "f64" else 1e-7)
