"""Masked rows around the limits that decide between their lists, launches and walks.

Multiplications and mask entries decide a row's list, the rows per list which
lists share a launch; A's rows and the longest row of B decide between groups of
lanes per B row and the flat walk.
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


def _check(A, B, M, dtype):
    import torch

    import paper_1801_03065_amd as spg

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


# mids: rows between the limits, 200 and 400 mask entries by turns (None: only the rows at the limits)
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m,mids", [(36, None), (16_384, None), (20_011, None), (65_537, None), (9_000, 8_192 - 48),
                                    (9_000, 8_192 + 1), (17_000, 8_192 + 1)])
def test_limits(m, mids, dtype):
    light, f_max, mw, mlong, mg = (_const(c) for c in ("MK_LIGHT", "MK_F", "MW_MAX", "MW_LONG", "MG_MAX"))
    assert (light % 64, f_max % 64) == (0, 0) and (_const("MK_MID_WG"), _const("MK_JOIN")) == (8_192, 16_384)
    rng = np.random.default_rng(m)
    lens_b = np.full(N, 64)
    lens_b[-2:] = 63, 65
    B = synth.random_csr(N, K, lens_b, 1)
    special = []  # (B rows of a row of A: limit - 1, limit, limit + 1 multiplications; mask entries)
    for limit in (light, f_max):
        for last in (N - 2, None, N - 1):
            for entries in (mw, mw + 1, mlong, mlong + 1, mg, mg + 1):
                rows = rng.permutation(N - 2)[:limit // 64]
                if last is not None:
                    rows[-1] = last
                special.append((np.sort(rows), entries))
                assert lens_b[rows].sum() == limit + {N - 2: -1, None: 0, N - 1: 1}[last]
    for i in range(mids or 0):
        rows = rng.permutation(N - 2)[:light // 64 + 1]
        special.append((np.sort(rows), (200, 400)[i % 2]))
    lens_a = np.where(rng.random(m) < 0.5, 0, 1)
    lens_m = rng.integers(0, 4, m)
    at = np.sort(rng.choice(m, len(special), replace=False))
    at[-1] = m - 1
    for i, (rows, entries) in zip(at, special):
        lens_a[i], lens_m[i] = len(rows), entries
    A = synth.random_csr(m, N, lens_a, 2)
    for i, (rows, _) in zip(at, special):
        A.col_idx[A.row_ptr[i]:A.row_ptr[i + 1]] = rows
    _check(A, B, synth.random_csr(m, K, lens_m, 3), dtype)


# `over`: A entries of the longest row (or, of all rows, on average) beyond those
# that fill the turns (0: groups; 1: by turns, or flat, for groups of 8 lanes and more)
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("longest", [1, 2, 4, 5, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("by,over", [("row", 0), ("row", 1), ("mean", 0), ("mean", 1)])
def test_groups(longest, by, over, dtype):
    turns = _const("MK_TURNS")
    m, n = 501, 3000
    rng = np.random.default_rng(longest)
    lens_b = rng.integers(0, longest + 1, n)
    lens_b[0] = longest
    B = synth.random_csr(n, K, lens_b, 1)
    full = turns * 64 // (1 << (longest - 1).bit_length())  # A entries of a row that fill the turns
    if by == "row":
        lens_a = rng.integers(0, full + 1, m)
        lens_a[-1] = full + over
    else:
        total = full * m + over
        lens_a = rng.multinomial(total // 2, np.full(m, 1 / m))
        lens_a[:8] = [0, 1, 63, 64, 65, 128, 129, 200]  # whole and partial chunks of 64 entries
        rest = total - lens_a.sum()
        while rest:  # spread what is left
            i = rng.integers(8, m)
            d = int(np.clip(rest, -lens_a[i], min(n - lens_a[i], 200)))
            lens_a[i] += d
            rest -= d
        assert lens_a.sum() == total
    M = synth.random_csr(m, K, rng.integers(0, 257, m), 3)
    _check(synth.random_csr(m, n, lens_a, 2), B, M, dtype)


def test_empty_b():
    # A's rows meet only empty rows of B, which has no entry at all
    A = synth.random_csr(70, 50, np.full(70, 9), 1)
    B = synth.random_csr(50, K, np.zeros(50, dtype=np.int64), 2)
    _check(A, B, synth.random_csr(70, K, np.full(70, 20), 3), "f64")
