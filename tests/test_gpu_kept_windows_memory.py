"""Memory of the heavy rows' kept bit windows: they yield to what a product needs."""
import numpy as np
import pytest

import synth
from helpers import check_f64, dev, oracle_ref, run

pytestmark = pytest.mark.gpu

K = 33_000  # 1032 window words a row
MB = 1 << 20


def _free():
    import torch

    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _column_times_row(m):
    """m rows of K products each: 4128 bytes of window per row."""
    A = synth.Csr(m, 1, np.arange(m + 1, dtype=np.int64), np.zeros(m, np.int32), np.arange(1.0, m + 1))
    return A, synth.Csr(1, K, np.array([0, K], np.int64), np.arange(K, dtype=np.int32), np.ones(K))


def _hog(leave):
    import torch

    return torch.empty(_free() - leave, dtype=torch.uint8, device="cuda")


def _panel_is_right(h, dA, dB, rows):
    import torch

    import paper_1801_03065_amd as spg

    ci = torch.full((rows * K,), -1, dtype=torch.int32, device="cuda")
    v = torch.zeros(rows * K, dtype=torch.float64, device="cuda")
    spg.spgemm_numeric_rows(h, dA, dB, 0, rows, ci, v)
    h.check_errors()
    assert torch.equal(ci.view(rows, K), torch.arange(K, device="cuda", dtype=torch.int32).expand(rows, K))
    assert torch.equal(v.view(rows, K), torch.arange(1.0, rows + 1, device="cuda", dtype=torch.float64)[:, None].expand(rows, K))


def test_given_back_when_a_plan_does_not_use_them():
    import torch

    import paper_1801_03065_amd as spg

    A, B = _column_times_row(70_000)
    h, dA, dB = spg.Handle(), dev(A), dev(B)
    start = _free()
    spg.spgemm_symbolic(h, dA, dB, torch.int64)
    assert start - _free() > 70_000 * 4128  # kept: 275 MiB
    _panel_is_right(h, dA, dB, 50)
    S = synth.laplace2d_5pt(30, 30)
    ref, mag = oracle_ref(S, S)
    got, _ = run(S, S, handle=h)
    check_f64(ref, mag, got)
    assert start - _free() < 100 * MB


def test_not_kept_where_memory_is_short():
    import torch

    import paper_1801_03065_amd as spg

    A, B = _column_times_row(70_000)
    h, dA, dB = spg.Handle(), dev(A), dev(B)
    hog = _hog(3072 * MB)
    try:
        start = _free()
        spg.spgemm_symbolic(h, dA, dB, torch.int64)
        assert start - _free() < 150 * MB
        _panel_is_right(h, dA, dB, 50)
    finally:
        del hog


def test_given_up_for_the_next_plan():
    """1.2 GB of windows are held when a plan of 12M rows needs more than what is free."""
    import torch

    import paper_1801_03065_amd as spg

    A, B = _column_times_row(300_000)
    h, dA, dB = spg.Handle(), dev(A), dev(B)
    start = _free()
    spg.spgemm_symbolic(h, dA, dB, torch.int64)
    assert start - _free() > 300_000 * 4128
    m = 12_000_000
    one = torch.ones(m, dtype=torch.float64, device="cuda")
    I = spg.DeviceCsr(m, m, torch.arange(m + 1, dtype=torch.int32, device="cuda"),
                      torch.arange(m, dtype=torch.int32, device="cuda"), one)
    hog = _hog(100 * MB)
    try:
        rp, nnz = spg.spgemm_symbolic(h, I, I)
        assert nnz == m and torch.equal(rp, I.row_ptr)
    finally:
        del hog


@pytest.mark.parametrize("rows,wide", [(1020, 1020), (1030, 1030), (1030, 1)])
def test_room_by_the_bound_and_by_the_exact_size(rows, wide):
    """Rows times the widest window (32768 words) below 2^25 words, past it, and past it for one wide row only."""
    import torch

    n, lb, na, k = 400, 512, 66, 1 << 20
    assert (rows * 32_768 > 1 << 25) == (rows > 1024)
    B = synth.random_csr(n, k, np.full(n, lb), 1)
    N = synth.random_csr(n, 90_000, np.full(n, lb), 2)  # B's second half: a narrow window
    B = synth.Csr(2 * n, k, np.concatenate([B.row_ptr, B.nnz + N.row_ptr[1:]]), np.concatenate([B.col_idx, N.col_idx]),
                  np.concatenate([B.values, N.values]))
    for r in range(n):  # both ends of the window in every wide row
        B.col_idx[B.row_ptr[r]], B.col_idx[B.row_ptr[r + 1] - 1] = 0, k - 1
    rng = np.random.default_rng(3)
    ci = np.stack([np.sort(rng.choice(n, na, replace=False)) + (0 if i < wide else n) for i in range(rows)])
    A = synth.Csr(rows, 2 * n, np.arange(0, rows * na + 1, na, dtype=np.int64), ci.reshape(-1).astype(np.int32),
                  rng.standard_normal(rows * na))
    ref, S = oracle_ref(A, B)
    got, h = run(A, B)
    assert h.stats()["rows_numeric"]["dense_wg"] == rows
    check_f64(ref, S, got)
    torch.cuda.empty_cache()
