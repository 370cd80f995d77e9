"""New values on a known structure, rows of every size class and several chunks of A entries, against the oracle."""
import numpy as np
import pytest

import synth
from helpers import check_f32, check_f64, dev, f32_inputs, oracle_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,opts", [("f64", {}), ("f32", {}), ("f32", {"fp32_mode": 1}), ("f32", {"fp32_mode": 2})])
@pytest.mark.parametrize("k", [2_000, 60_000, 3_000_000])
def test_values_on_maps(dtype, opts, k):
    import torch

    import paper_1801_03065_amd as spg

    rng = np.random.default_rng(k)
    n = 400
    lens = rng.choice([0, 1, 3, 16, 40], n)  # empty B rows inside the runs
    lens[:64] = 16  # A rows of 4 to 64 of these: 64, ..., 1024 multiplications exactly
    B = synth.random_csr(n, k, lens, k + 1)
    cols = [np.arange(c) for c in (4, 5, 8, 9, 16, 17, 32, 33, 63, 64)] * 2
    cols += [np.sort(rng.choice(n, c, replace=False)) for c in (0, 1, 7, 64, 65, 100, 128, 129, 200) for _ in range(3)]
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    A = synth.Csr(len(cols), n, rp, np.concatenate(cols).astype(np.int32), rng.standard_normal(int(rp[-1])))
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
    else:  # at most 200 products an entry: gamma_200 for plain sums, one rounding and FP64's for the others
        check_f32(ref, S, got, rel=201 * 2.0**-24 * 1.01 if not opts else 6.1e-8)
