"""A symbolic call that is refused leaves the caller's row pointers as they were."""
import ctypes

import numpy as np
import pytest

import synth
from helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k", [(70_000, 33_000), (1_100_000, 2_000)])  # heavy rows, bit-window rows
def test_row_pointers_after_index_overflow(m, k):
    """A column of ones times a full row: m * k > 2^31 entries do not fit an int32 row_ptr."""
    import torch

    import paper_1801_03065_amd as spg

    assert m * k > 2 ** 31
    A = synth.Csr(m, 1, np.arange(m + 1, dtype=np.int64), np.zeros(m, np.int32), np.ones(m))
    B = synth.Csr(1, k, np.array([0, k], np.int64), np.arange(k, dtype=np.int32), np.ones(k))
    h, dA, dB = spg.Handle(), dev(A), dev(B)
    rp = torch.full((m + 1,), -77, dtype=torch.int32, device="cuda")
    nnz = ctypes.c_int64(-5)
    a, b = spg._csr(dA), spg._csr(dB)
    st = spg.lib().spgemm_symbolic(h.ptr, ctypes.byref(a), ctypes.byref(b), ctypes.c_void_p(rp.data_ptr()),
                                   spg.SPG_I32, ctypes.byref(nnz))
    assert st == spg.SPG_ERR_INDEX_OVERFLOW and nnz.value == -5
    assert bool((rp == -77).all())
    rp64, n = spg.spgemm_symbolic(h, dA, dB, torch.int64)
    assert n == m * k and torch.equal(rp64, torch.arange(m + 1, device="cuda") * k)
