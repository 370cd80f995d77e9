"""Short rows (up to 64 products, teams of 8 to 64 lanes) against the oracle: every team size, repeated columns,
A rows longer than the team, and matrices too wide for a packed (column, lane) key."""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, f32_inputs, oracle_ref, run

pytestmark = pytest.mark.gpu


def _product(fmax, k, seed, pool):
    """Rows of 0 to fmax products; B rows of 0, 1, 2, 5 or 16 columns out of the first `pool` and the last columns."""
    rng = np.random.default_rng(seed)
    n = 500
    lens = rng.choice([0, 0, 1, 2, 5, 16], n)
    near = np.unique(np.concatenate([np.arange(min(pool, k)), np.arange(max(0, k - pool), k)]))
    cols = [np.sort(rng.choice(near, c, replace=False)) for c in lens]
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    B = synth.Csr(n, k, rp, np.concatenate(cols).astype(np.int32), rng.standard_normal(int(rp[-1])))
    empty, rows = np.flatnonzero(lens == 0), []
    for r in range(400):
        want = [fmax, fmax - 1, 1, int(rng.integers(0, fmax + 1))][r % 4]
        take, f = [], 0
        for c in rng.permutation(n):
            if lens[c] and f + lens[c] <= want:
                take.append(c)
                f += lens[c]
        if r % 7 == 0:  # more A entries than lanes: most of their B rows are empty
            take += list(empty[:150])
        rows.append(np.sort(np.unique(take)).astype(np.int64))
    arp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    return synth.Csr(len(rows), n, arp, np.concatenate(rows).astype(np.int32), rng.standard_normal(int(arp[-1]))), B


@pytest.mark.parametrize("k", [40, 5000, 1 << 26, (1 << 26) + 1])
@pytest.mark.parametrize("fmax", [8, 9, 32, 64])
def test_teams(fmax, k):
    for pool in (20, 2000) if k < 1 << 20 else (20,):  # many and few repeats
        A, B = _product(fmax, k, fmax + k % 97, pool)
        ref, S = oracle_ref(A, B)
        got, h = run(A, B)
        check_f64(ref, S, got)
        st = h.stats()["rows_numeric"]
        assert st["short_rows"] + st["empty"] == A.nrows


@pytest.mark.parametrize("opts", [{}, {"fp32_mode": 1}, {"fp32_mode": 2}])
@pytest.mark.parametrize("k", [40, 100_000_000])
def test_fp32(opts, k):
    A, B = _product(64, k, 5, 20)
    A, B = f32_inputs(A), f32_inputs(B)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, B, dtype="f32", **opts)
    # at most 64 products an entry: gamma_64 for plain sums, one rounding and FP64's for the others
    check_f32(ref, S, got, rel=65 * 2.0**-24 * 1.01 if not opts else 6.1e-8)


def test_one_product_per_a_entry():
    """B rows of at most one entry, A rows of up to 64 entries: no expansion; repeated columns between them."""
    rng = np.random.default_rng(2)
    n = 300
    lens = rng.choice([0, 1, 1, 1], n)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    B = synth.Csr(n, 30, rp, rng.integers(0, 30, int(rp[-1])).astype(np.int32), rng.standard_normal(int(rp[-1])))
    A = synth.random_csr(200, n, rng.integers(0, 65, 200), 4)
    ref, S = oracle_ref(A, B)
    got, _ = run(A, B)
    check_f64(ref, S, got)
