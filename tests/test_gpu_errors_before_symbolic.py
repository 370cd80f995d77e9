"""check_errors on a handle without a symbolic phase: nothing has gone wrong yet."""
import ctypes

import numpy as np
import pytest

import synth
from helpers import dev

pytestmark = pytest.mark.gpu


def test_check_errors_first():
    import torch

    import paper_1801_03065_amd as spg

    A = synth.random_csr(20, 20, np.full(20, 3), 1)
    d = dev(A, "f64")
    hip = spg.lib()  # the runtime's functions by way of the library that links it
    dirt = []
    for size in [1 << s for s in range(8, 17)] * 32:  # small blocks that a new handle is likely to get
        p = ctypes.c_void_p()
        assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(size)) == 0
        assert hip.hipMemset(p, 7, ctypes.c_size_t(size)) == 0
        dirt.append(p)
    torch.cuda.synchronize()
    for p in dirt:
        assert hip.hipFree(p) == 0
    for _ in range(16):
        h = spg.Handle()
        h.check_errors()
        spg.spgemm_masked(h, d, d, d)
        h.check_errors()
