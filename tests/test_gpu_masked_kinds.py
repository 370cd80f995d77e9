"""Masked products at the edges of the row kinds: mask rows of 256 / 257 and
2048 / 2049 entries, rows around 8192 multiplications, A rows beyond one chunk
of 512 entries, few and many rows whose table lies in HBM, 32- and 64-bit
product numbers (B from 4.2M entries on), columns out of range."""
import numpy as np
import pytest

import oracle
import synth
from helpers import dev, f32_inputs

pytestmark = pytest.mark.gpu


def _masked(A, B, M, structural=False, dtype="f64"):
    import torch

    import paper_1801_03065_amd as spg

    out = spg.spgemm_masked(spg.Handle(), dev(A, dtype), dev(B, dtype), dev(M, dtype), structural=structural)
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def _check(A, B, M, dtype="f64"):
    A0, B0 = (A, B) if dtype == "f64" else (f32_inputs(A), f32_inputs(B))
    want, S = oracle.masked(A0, B0, M, with_abs=True)
    got = _masked(A, B, M, dtype=dtype)
    # FP32 inputs: exact products summed in FP64, one rounding of the result
    tol = 1e-12 * np.maximum(np.abs(want), S) if dtype == "f64" else 2.0 ** -24 * np.abs(want) + 1e-12 * S
    assert np.all(np.abs(got - want) <= tol)
    assert np.array_equal(_masked(A, B, M, structural=True, dtype=dtype), oracle.masked(A, B, M, structural=True))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_kind_edges(dtype):
    lens_m = np.array([0, 1, 2, 255, 256, 257, 300, 2047, 2048, 2049, 3000, 5000] * 2)
    lens_a = np.repeat([20, 700], 12)  # about 800 and 28,000 multiplications a row
    m, n, k = lens_m.size, 900, 6000
    A = synth.shuffle_columns(synth.random_csr(m, n, lens_a, 1), 2)
    B = synth.shuffle_columns(synth.random_csr(n, k, np.random.default_rng(3).integers(0, 80, n), 4), 5)
    M = synth.shuffle_columns(synth.random_csr(m, k, lens_m, 6), 7)
    _check(A, B, M, dtype)


def test_multiplications_around_the_wavefront_limit():
    lens_a = np.array([63, 64, 65, 128, 1, 0])  # times 128 entries per row of B: 8064 .. 16384
    A = synth.random_csr(6, 300, lens_a, 1)
    B = synth.random_csr(300, 5000, np.full(300, 128), 2)
    M = synth.random_csr(6, 5000, np.full(6, 200), 3)
    _check(A, B, M)


def test_many_rows_with_tables_in_hbm():
    """More such rows than workgroups: a slice per workgroup, not per row."""
    m, n, k = 700, 40, 2600
    A = synth.random_csr(m, n, np.full(m, 10), 1)
    B = synth.random_csr(n, k, np.full(n, 90), 2)
    M = synth.random_csr(m, k, np.full(m, 2100), 3)
    _check(A, B, M)


def test_64_bit_product_numbers():
    n, per = 4300, 1000
    B = synth.random_csr(n, 100_000, np.full(n, per), 1)
    A = synth.random_csr(40, n, np.random.default_rng(2).integers(1, 60, 40), 2)
    M = synth.random_csr(40, 100_000, np.tile([100, 400, 2500, 250], 10), 3)
    assert B.nnz * 512 >= 2 ** 31
    _check(A, B, M)


@pytest.mark.parametrize("where", ["A", "M"])
def test_column_out_of_range_is_refused(where):
    import paper_1801_03065_amd as spg

    A = synth.random_csr(30, 40, np.full(30, 5), 1)
    B = synth.random_csr(40, 50, np.full(40, 5), 2)
    M = synth.random_csr(30, 50, np.full(30, 5), 3)
    bad = A if where == "A" else M
    bad.col_idx[-1] = bad.ncols
    with pytest.raises(spg.SpgemmError):
        _masked(A, B, M)
