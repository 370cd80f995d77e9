"""New values on maps where B's rows have a few entries: a chunk of 64 A entries on one lane per
B row, or flat as soon as one of its B rows is longer, against the oracle."""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, dev, f32_inputs, oracle_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,opts", [("f64", {}), ("f32", {}), ("f32", {"fp32_mode": 1}), ("f32", {"fp32_mode": 2})])
@pytest.mark.parametrize("longest", [1, 2, 3])
def test_values(dtype, opts, longest):
    import torch

    import paper_1801_03065_amd as spg

    rng = np.random.default_rng(longest)
    n, k = 2_500, 60_000
    lens = rng.integers(0, longest + 1, n)  # empty B rows too
    lens[n // 2:] = np.minimum(lens[n // 2:], 2)  # chunks with and without the longest
    B = synth.random_csr(n, k, lens, longest + 1)
    sizes = [0, 1, 2, 31, 63, 64, 65, 127, 128, 129, 200, 640, 1000, 1800] * 4  # every kind of row that has a map
    A = synth.random_csr(len(sizes), n, np.array(sizes), 7)
    A2 = synth.revalue(A, 3)
    if dtype == "f32":
        A, A2, B = f32_inputs(A), f32_inputs(A2), f32_inputs(B)
    h = spg.Handle(**opts)
    td = torch.float64 if dtype == "f64" else torch.float32
    dA, dB = dev(A, dtype), dev(B, dtype)
    rpc, nnz = spg.spgemm_symbolic(h, dA, dB)
    C = spg.spgemm_numeric(h, dA, dB, rpc, nnz)
    d2 = dA.with_values(torch.as_tensor(A2.values, device="cuda").to(td))
    for _ in range(2):  # the second call finds the maps built
        C.values.fill_(float("nan"))
        spg.spgemm_numeric_values(h, d2, dB, C)
    h.check_errors()
    ref, S = oracle_ref(A2, B)
    got = (rpc.cpu().numpy().astype(np.int64), C.col_idx.cpu().numpy(), C.values.cpu().numpy())
    if dtype == "f64":
        check_f64(ref, S, got)
    else:  # at most 1800 products an entry: gamma_1800 for plain sums, one rounding and FP64's for the others
        check_f32(ref, S, got, rel=1801 * 2.0**-24 * 1.01 if not opts else 6.1e-8)
