"""Masked rows around the multiplications that decide between a wavefront and a workgroup.

The limit depends on the mask's rows (few rows: the lower one), as does the
number of rows that 16 lanes classify one after the other.
"""
import os
import re

import numpy as np
import pytest

import oracle
import synth
from helpers import dev, f32_inputs

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1801_03065_amd", "csrc")
K, N = 5000, 400  # B: rows of 64 columns, then one of 63 and one of 65


def _const(name):
    for f in ("spg_masked.hip", "spg_internal.hpp"):
        m = re.search(rf"\b{name} = (\d+)", open(os.path.join(CSRC, f)).read())
        if m:
            return int(m.group(1))
    raise KeyError(name)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m", [9, 16_384, 20_011, 32_768, 32_769, 40_003])
def test_limits(m, dtype):
    import torch

    import paper_1801_03065_amd as spg

    few, f_few, f_max = _const("MK_FEW"), _const("MK_F_FEW"), _const("MK_F")
    assert (few, f_few % 64, f_max % 64) == (32_768, 0, 0)  # the sizes below lie around these
    rng = np.random.default_rng(m)
    lens_b = np.full(N, 64)
    lens_b[-2:] = 63, 65
    B = synth.random_csr(N, K, lens_b, 1)
    special = []  # B rows of a row of A: limit - 1, limit, limit + 1 multiplications
    for limit in (f_few, f_max):
        for last in (N - 2, None, N - 1):
            rows = rng.permutation(N - 2)[:limit // 64 - 1]
            special.append(np.sort(np.append(rows, last if last is not None else np.setdiff1d(np.arange(N - 2), rows)[0])))
            assert lens_b[special[-1]].sum() == limit + {N - 2: -1, None: 0, N - 1: 1}[last]
    lens_a = np.where(rng.random(m) < 0.5, 0, 1)
    lens_m = rng.integers(0, 4, m)
    at = np.sort(rng.choice(m, len(special), replace=False))
    at[-1] = m - 1
    for i, rows in zip(at, special):
        lens_a[i], lens_m[i] = len(rows), 200
    A = synth.random_csr(m, N, lens_a, 2)
    for i, rows in zip(at, special):
        A.col_idx[A.row_ptr[i]:A.row_ptr[i + 1]] = rows
    M = synth.random_csr(m, K, lens_m, 3)
    dA, dB, dM = dev(A, dtype), dev(B, dtype), dev(M, dtype)
    h = spg.Handle()
    got = spg.spgemm_masked(h, dA, dB, dM)
    count = spg.spgemm_masked(h, dA, dB, dM, structural=True)
    torch.cuda.synchronize()
    assert np.array_equal(count.cpu().numpy().astype(np.float64), oracle.masked(A, B, M, structural=True))
    A0, B0 = (A, B) if dtype == "f64" else (f32_inputs(A), f32_inputs(B))
    want, S = oracle.masked(A0, B0, M, with_abs=True)
    tol = 1e-12 * np.maximum(np.abs(want), S) if dtype == "f64" else 2.0 ** -24 * np.abs(want) + 1e-12 * S
    assert np.all(np.abs(got.cpu().numpy().astype(np.float64) - want) <= tol)
