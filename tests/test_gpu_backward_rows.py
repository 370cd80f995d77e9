"""Backward at the edges of its kernel: C rows at the LDS limit (2047 / 2048
entries) and beyond, A rows of one and several chunks of 64 entries, one and
several rounds of products, empty rows of A and B, and a B large enough for
64-bit product numbers."""
import numpy as np
import pytest

import oracle
import synth
from helpers import dev, f32_inputs

pytestmark = pytest.mark.gpu


def _check(A, B, dtype):
    import torch

    import paper_1801_03065_amd as spg

    A0, B0 = (A, B) if dtype == "f64" else (f32_inputs(A), f32_inputs(B))
    C = oracle.spgemm(A0, B0)
    G = np.random.default_rng(5).standard_normal(C.nnz).astype(np.float32).astype(np.float64)
    h = spg.Handle()
    dA_, dB_ = dev(A, dtype), dev(B, dtype)
    rp, nnz = spg.spgemm_symbolic(h, dA_, dB_, torch.int64)
    Cd = spg.spgemm_numeric(h, dA_, dB_, rp, nnz)
    Gd = spg.DeviceCsr(A.nrows, B.ncols, rp, Cd.col_idx, torch.as_tensor(G, device="cuda").to(Cd.values.dtype))
    dA, dB = spg.spgemm_backward(h, dA_, dB_, Gd)
    h.check_errors()
    rdA, rdB = oracle.grad(A0, B0, C, G)
    sA, sB = oracle.grad(A0.with_values(np.abs(A0.values)), B0.with_values(np.abs(B0.values)), C, np.abs(G))
    # FP32: dA is summed in FP64 and rounded once; dB sums up to nnz of a column of A rounded products
    tA = 1e-12 if dtype == "f64" else 2.0 ** -23
    tB = 1e-12 if dtype == "f64" else 2.0 ** -24 * (np.bincount(A.col_idx, minlength=1).max() + 2)
    assert np.all(np.abs(dA.cpu().numpy() - rdA) <= tA * np.maximum(sA, 1e-300))
    assert np.all(np.abs(dB.cpu().numpy() - rdB) <= tB * np.maximum(sB, 1e-300))
    return C


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_row_lengths_around_the_lds_limit(dtype):
    """C rows of exactly 2046 .. 2049 and 5000 entries: B rows tile the columns, a row of A takes some of them."""
    per = np.concatenate([np.full(40, 50), [46, 1, 1, 1, 1], np.full(60, 50)])
    k = int(per.sum())
    rp = np.concatenate([[0], np.cumsum(per)])
    rng = np.random.default_rng(3)
    B = synth.Csr(per.size, k, rp, np.arange(k, dtype=np.int32), rng.standard_normal(k))
    rows = [np.arange(41), np.arange(42), np.arange(43), np.arange(44), np.arange(105), np.array([], int), np.array([40])]
    A = synth.Csr(len(rows), per.size, np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64),
                  np.concatenate(rows).astype(np.int32), rng.standard_normal(sum(len(r) for r in rows)))
    C = _check(A, B, dtype)
    assert list(C.row_lengths()[:5]) == [2046, 2047, 2048, 2049, k]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("la,lb", [(3, 2), (64, 2), (65, 2), (130, 9), (20, 64), (63, 65), (200, 90)])
def test_chunks_and_rounds(la, lb, dtype):
    rng = np.random.default_rng(la + lb)
    lens = rng.integers(0, la + 1, 60)
    lens[::7] = la
    A = synth.shuffle_columns(synth.random_csr(60, 300, lens, la), 1)
    B = synth.shuffle_columns(synth.random_csr(300, 700, rng.integers(0, lb + 1, 300), lb), 2)
    _check(A, B, dtype)


def test_64_bit_product_numbers():
    n, per = 33_600, 1000
    B = synth.Csr(n, 4000, np.arange(0, n * per + 1, per, dtype=np.int64),
                  (np.arange(per, dtype=np.int32)[None, :] + (np.arange(n, dtype=np.int32) % 3000)[:, None]).reshape(-1),
                  np.random.default_rng(1).standard_normal(n * per))
    A = synth.random_csr(12, n, np.full(12, 70), 2)
    assert B.nnz * 64 >= 2 ** 31
    _check(A, B, "f64")
