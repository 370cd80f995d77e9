"""Performance cases of the two-phase SpGEMM library: the products a user runs, through the package's public calls.

Every case is a family with sizes. Inputs are generated on the GPU: the structure of a matrix belongs to the case (as
that of a mesh or a graph file does), its values come from the seed; the graph of a triangle count is one of the seed's
own. `run` is one pass of a user's program and returns whole outputs, `exact` gives the same values from plain torch in
FP64.

Families
  stencil   A*A of a 2D 5-point, 3D 7-point or 3D 27-point operator with variable coefficients (PDE codes)
  galerkin  the multigrid coarse operator P^T*(A*P) with 2x2x2 aggregation on a 27-point operator
  random    A*B of random sparse matrices, Poisson row sizes, B optionally with unsorted rows
  rmat      A*A of a symmetric R-MAT graph (power-law rows)
  batch     many independent random products under one plan
  triangles triangle counting, L*L on the pattern of L, of an R-MAT graph; or the same product with values
  train     one forward and backward of a differentiable product, 7-point operator times a random matrix

Modes of the first four and of batch: "full" runs both phases, "numeric" the numeric phase on a kept plan with new
values, "values" the numeric phase on a known structure (the columns are in place).
"""
import torch

import paper_1801_03065_amd as spg

DTYPES = {"f64": torch.float64, "f32": torch.float32}


# ------------------------------------------------------------------ cases
def listed():
    return [
        # a small PDE product in a time step or a coarse multigrid level: latency and launches count
        {"name": "laplace5_64", "family": "stencil", "points": 5, "g": 64, "mode": "full", "dtype": "f64"},
        # the benchmark's stencil square, first time on a structure
        {"name": "stencil27_100", "family": "stencil", "points": 27, "g": 100, "mode": "full", "dtype": "f64"},
        # an odd grid in FP32, new coefficients on a kept plan (time stepping, nonlinear solves)
        {"name": "stencil27_61_reuse_f32", "family": "stencil", "points": 27, "g": 61, "mode": "numeric",
         "dtype": "f32"},
        # the benchmark's multigrid setup product
        {"name": "galerkin_100", "family": "galerkin", "g": 100, "mode": "full", "dtype": "f64"},
        # a mid-size general product whose B comes with its rows in no order
        {"name": "random_20011_unsorted", "family": "random", "n": 20011, "k": 20011, "lam": 12.0, "unsorted": True,
         "rp64": False, "mode": "full", "dtype": "f64"},
        # large, very sparse, columns over a wide range, 64-bit row pointers
        {"name": "random_1500k_wide", "family": "random", "n": 1500000, "k": 1500000, "lam": 7.0, "unsorted": False,
         "rp64": True, "mode": "full", "dtype": "f64"},
        # a power-law graph square, both phases
        {"name": "rmat_17", "family": "rmat", "scale": 17, "mode": "full", "dtype": "f64"},
        # a smaller graph in FP32, new weights on a kept plan
        {"name": "rmat_15_reuse_f32", "family": "rmat", "scale": 15, "mode": "numeric", "dtype": "f32"},
        # the batch form, first time on its structures
        {"name": "batch_48", "family": "batch", "count": 48, "n_hi": 65536, "mode": "full", "dtype": "f64"},
        # the batch form with new values on known structures
        {"name": "batch_48_values_f32", "family": "batch", "count": 48, "n_hi": 65536, "mode": "values",
         "dtype": "f32"},
        # graph analytics: triangles of a power-law graph
        {"name": "triangles_18", "family": "triangles", "scale": 18, "structural": True, "dtype": "f64"},
        # training through a sparse product
        {"name": "train_64_f32", "family": "train", "g": 64, "per_row": 16, "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    family = rng.choice(["stencil", "stencil", "galerkin", "random", "random", "rmat", "rmat", "batch", "triangles",
                         "train"])
    dtype = rng.choice(["f64", "f64", "f32"])
    mode = rng.choice(["full", "full", "numeric", "values"])
    if family == "stencil":
        points = rng.choice([5, 7, 27])
        g = _log_int(rng, 24, 1000) if points == 5 else _log_int(rng, 9, 100)
        return {"family": family, "points": points, "g": g, "mode": mode, "dtype": dtype}
    if family == "galerkin":
        return {"family": family, "g": 2 * _log_int(rng, 5, 50), "mode": "full", "dtype": dtype}
    if family == "random":
        lam = round(rng.uniform(4.0, 32.0), 2)
        n = _log_int(rng, 1000, int(1.2e8 / (lam * lam)))  # at most about 1.2e8 multiplications
        k = max(200, int(n * rng.choice([0.25, 1.0, 1.0, 3.0])))
        return {"family": family, "n": n, "k": k, "lam": lam, "unsorted": rng.random() < 0.4,
                "rp64": rng.random() < 0.3, "mode": mode, "dtype": dtype}
    if family == "rmat":
        return {"family": family, "scale": rng.randint(10, 16), "mode": mode, "dtype": dtype}
    if family == "batch":
        return {"family": family, "count": _log_int(rng, 2, 40), "n_hi": _log_int(rng, 2000, 65536),
                "mode": rng.choice(["full", "numeric", "values"]), "dtype": dtype}
    if family == "triangles":
        return {"family": family, "scale": rng.randint(11, 18), "structural": rng.random() < 0.6, "dtype": dtype}
    return {"family": "train", "g": _log_int(rng, 9, 64), "per_row": rng.randint(4, 16), "dtype": dtype}


# ------------------------------------------------------------------ inputs (GPU, from the seed alone)
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _shape_gen(*sizes):
    """The generator of a structure: the same for the same sizes."""
    h = 1
    for s in sizes:
        h = (h * 1000003 + int(1000 * s)) % (1 << 40)
    return _gen(h)


def _csr(nrows, ncols, rows, cols, values, dtype, rp64=False):
    """CSR from entries grouped by row."""
    rp = torch.zeros(nrows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(torch.bincount(rows, minlength=nrows), 0, out=rp[1:])
    return spg.DeviceCsr(nrows, ncols, rp if rp64 else rp.to(torch.int32), cols.to(torch.int32).contiguous(),
                         values.to(dtype).contiguous())


def _normal(g, n):
    return torch.randn(n, generator=g, device="cuda", dtype=torch.float64)


def _uniform(g, n):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _stencil(points, size, g, dtype):
    """Operator on a size^2 (5 points) or size^3 (7, 27 points) grid: off-diagonals around -1, diagonal around their
    number, each varied by up to a tenth."""
    dim = 2 if points == 5 else 3
    offs = [(dz, dy, dx) for dz in ((0,) if dim == 2 else (-1, 0, 1)) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
    if points != 27:
        offs = [o for o in offs if sum(map(abs, o)) <= 1]
    n = size ** dim
    p = torch.arange(n, device="cuda")
    x, y, z = p % size, (p // size) % size, p // (size * size)
    cols = torch.empty(n, len(offs), dtype=torch.int64, device="cuda")
    for s, (dz, dy, dx) in enumerate(offs):  # increasing column order
        ok = (x + dx >= 0) & (x + dx < size) & (y + dy >= 0) & (y + dy < size)
        if dim == 3:
            ok &= (z + dz >= 0) & (z + dz < size)
        cols[:, s] = torch.where(ok, p + (dz * size + dy) * size + dx, -1)
    ok = cols >= 0
    rows = p.unsqueeze(1).expand(n, len(offs))[ok]
    cols = cols[ok]
    values = torch.where(rows == cols, float(points - 1), -1.0) * (1.0 + 0.1 * _uniform(g, cols.numel()))
    return _csr(n, n, rows, cols, values, dtype)


def _random(n, k, lam, which, g, dtype, unsorted=False, rp64=False):
    """n x k, Poisson(lam) uniform columns per row (repeats dropped), N(0, 1) values; `which`: 0 for A, 1 for B."""
    sg = _shape_gen(n, k, lam, which)
    counts = torch.poisson(torch.full((n,), float(lam), device="cuda"), generator=sg).to(torch.int64)
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), counts)
    cols = torch.randint(0, k, (rows.numel(),), generator=sg, device="cuda")
    keys = torch.unique(rows * k + cols)
    rows, cols = keys // k, keys % k
    if unsorted:
        order = torch.argsort(rows.double() + _uniform(sg, rows.numel()))
        rows, cols = rows[order], cols[order]
    return _csr(n, k, rows, cols, _normal(g, cols.numel()), dtype, rp64)


def _rmat_edges(scale, g):
    """Undirected edges (lo, hi) of an R-MAT graph, 16 * 2^scale draws with (0.57, 0.19, 0.19, 0.05)."""
    n, a, b, c = 1 << scale, 0.57, 0.19, 0.19
    u = torch.zeros(16 * n, dtype=torch.int64, device="cuda")
    v = torch.zeros_like(u)
    for bit in range(scale):
        r = torch.rand(u.numel(), generator=g, device="cuda")
        u |= (r >= a + b).to(torch.int64) << bit
        v |= (((r >= a) & (r < a + b)) | (r >= a + b + c)).to(torch.int64) << bit
    keep = u != v
    lo, hi = torch.minimum(u, v)[keep], torch.maximum(u, v)[keep]
    keys = torch.unique(lo * n + hi)
    return n, keys // n, keys % n


def _rmat(scale, g, dtype):
    n, lo, hi = _rmat_edges(scale, _shape_gen(scale))
    w = 2.0 * _uniform(g, lo.numel()) - 1.0
    keys, order = torch.sort(torch.cat([lo * n + hi, hi * n + lo]))
    return _csr(n, n, keys // n, keys % n, torch.cat([w, w])[order], dtype)


def _aggregation(size, dtype):
    """Piecewise-constant prolongator P of 2x2x2 aggregates on a size^3 grid (size even), and its transpose."""
    h, n = size // 2, size ** 3
    p = torch.arange(n, device="cuda")
    x, y, z = p % size, (p // size) % size, p // (size * size)
    agg = ((z // 2) * h + y // 2) * h + x // 2
    one = torch.ones(n, device="cuda")
    order = torch.argsort(agg, stable=True)
    return _csr(n, h ** 3, p, agg, one, dtype), _csr(h ** 3, n, agg[order], order, one, dtype)


def _batch(count, n_hi, seed, dtype):
    """Operands of a batch, each side's columns and values back to back: n from 1000 to n_hi, mean row sizes 4 to 32."""
    u = torch.rand(2, count, generator=torch.Generator().manual_seed(count * 1000003 + n_hi))  # shapes: the case's
    g = _gen(seed)
    sides = ([], [])
    for i in range(count):
        n, lam = 1000 + int(float(u[0, i]) * (n_hi - 1000)), 4.0 + 28.0 * float(u[1, i])
        for which, side in enumerate(sides):
            side.append(_random(n, n, lam, 2 * i + which, g, dtype))
    packed = []
    for side in sides:
        ci, va = torch.cat([M.col_idx for M in side]), torch.cat([M.values for M in side])
        off, out = 0, []
        for M in side:
            out.append(spg.DeviceCsr(M.nrows, M.ncols, M.row_ptr, ci[off:off + M.nnz], va[off:off + M.nnz]))
            off += M.nnz
        packed.append(out)
    return packed


def _operands(case, seed):
    """The operands of a single product (A, B)."""
    g, dtype = _gen(seed), DTYPES[case["dtype"]]
    if case["family"] == "stencil":
        A = _stencil(case["points"], case["g"], g, dtype)
        return A, A
    if case["family"] == "random":
        A = _random(case["n"], case["n"], case["lam"], 0, g, dtype, rp64=case["rp64"])
        return A, _random(case["n"], case["k"], case["lam"], 1, g, dtype, case["unsorted"], case["rp64"])
    if case["family"] == "rmat":
        A = _rmat(case["scale"], g, dtype)
        return A, A
    if case["family"] == "triangles":
        n, lo, hi = _rmat_edges(case["scale"], g)
        some = torch.randperm(lo.numel(), generator=g, device="cuda")[:10 * n]  # 10 edges a vertex, whatever the seed
        keys, _ = torch.sort(hi[some] * n + lo[some])
        L = _csr(n, n, keys // n, keys % n, _normal(g, keys.numel()), dtype)
        return L, L
    A = _stencil(7, case["g"], g, dtype)  # train
    n = A.ncols
    return A, _random(n, n, case["per_row"], 1, g, dtype)


def prepare(case, seed):
    f, dtype = case["family"], DTYPES[case["dtype"]]
    st = {"case": case, "h": spg.Handle()}
    if f == "galerkin":
        st["A"] = _stencil(27, case["g"], _gen(seed), dtype)
        st["P"], st["Pt"] = _aggregation(case["g"], dtype)
        st["h2"] = spg.Handle()
        return st
    if f == "batch":
        st["As"], st["Bs"] = _batch(case["count"], case["n_hi"], seed, dtype)
        if case["mode"] != "full":
            rps, nnzs = spg.spgemm_batch_symbolic(st["h"], st["As"], st["Bs"])
            st["Cs"] = spg.batch_outputs(st["As"], st["Bs"], rps, nnzs, dtype)
            if case["mode"] == "values":
                spg.spgemm_batch_numeric(st["h"], st["As"], st["Bs"], st["Cs"])
        return st
    A, B = st["A"], st["B"] = _operands(case, seed)
    if f == "train":
        st["prod"] = spg.SparseProduct(A, B, handle=st["h"])
        st["a"] = A.values.clone().requires_grad_()
        st["b"] = B.values.clone().requires_grad_()
        st["grad"] = _normal(_gen(seed + 1000003), st["prod"].nnz).to(dtype)
    elif f != "triangles" and case["mode"] != "full":
        rp, nnz = spg.spgemm_symbolic(st["h"], A, B, rp_dtype=A.row_ptr.dtype)
        st["rp"], st["nnz"] = rp, nnz
        ci = torch.empty(nnz, dtype=torch.int32, device="cuda")
        st["C"] = spg.DeviceCsr(A.nrows, B.ncols, rp, ci, torch.empty(nnz, dtype=dtype, device="cuda"))
        if case["mode"] == "values":
            spg.spgemm_numeric(st["h"], A, B, rp, nnz, out=st["C"])
    return st


# ------------------------------------------------------------------ one pass
def _out(C):
    return {"row_ptr": C.row_ptr, "col_idx": C.col_idx, "values": C.values}


def run(state):
    case, h = state["case"], state["h"]
    f = case["family"]
    if f == "galerkin":
        AP = spg.spgemm(state["A"], state["P"], handle=h)
        return {"AP": _out(AP), "coarse": _out(spg.spgemm(state["Pt"], AP, handle=state["h2"]))}
    if f == "batch":
        As, Bs = state["As"], state["Bs"]
        if case["mode"] == "full":
            rps, nnzs = spg.spgemm_batch_symbolic(h, As, Bs)
            Cs = spg.spgemm_batch_numeric(h, As, Bs, spg.batch_outputs(As, Bs, rps, nnzs, As[0].values.dtype))
        elif case["mode"] == "numeric":
            Cs = spg.spgemm_batch_numeric(h, As, Bs, state["Cs"])
        else:
            Cs = spg.spgemm_batch_numeric_values(h, As, Bs, state["Cs"])
        total = sum(C.nnz for C in Cs)  # the products lie back to back: their entries as two whole arrays
        return {"col_idx": Cs[0].col_idx.as_strided((total,), (1,)), "values": Cs[0].values.as_strided((total,), (1,)),
                "row_ptr_first": Cs[0].row_ptr, "row_ptr_last": Cs[-1].row_ptr}
    A, B = state["A"], state["B"]
    if f == "triangles":
        return spg.spgemm_masked(h, A, B, A, structural=case["structural"])
    if f == "train":
        c = state["prod"](state["a"], state["b"])
        da, db = torch.autograd.grad(c, (state["a"], state["b"]), state["grad"])
        return {"c": c.detach(), "da": da, "db": db}
    if case["mode"] == "full":
        return _out(spg.spgemm(A, B, handle=h, rp_dtype=A.row_ptr.dtype))
    if case["mode"] == "numeric":
        return _out(spg.spgemm_numeric(h, A, B, state["rp"], state["nnz"], out=state["C"]))
    return _out(spg.spgemm_numeric_values(h, A, B, state["C"]))


# ------------------------------------------------------------------ what a pass cannot do without
def _bytes(M, values=True):
    return (M.row_ptr.element_size() * (M.nrows + 1) + M.nnz * (4 + (M.values.element_size() if values else 0)))


def _counts(A, B):
    """Multiplications and nnz(C) of A*B."""
    h = spg.Handle()
    _, nnz = spg.spgemm_symbolic(h, A, B, rp_dtype=torch.int64)
    return h.stats()["flops"], nnz


def work(case):
    """A and B read once, C written once, two operations per multiplication."""
    f = case["family"]
    vb = 8 if case["dtype"] == "f64" else 4
    if f == "galerkin":
        st = prepare(case, 0)
        A, P, Pt = st["A"], st["P"], st["Pt"]
        AP = spg.spgemm(A, P, handle=st["h"])
        f1, c1 = _counts(A, P)
        f2, c2 = _counts(Pt, AP)
        return {"bytes": _bytes(A) + _bytes(P) + 2 * _bytes(AP) + _bytes(Pt) + 4 * (Pt.nrows + 1) + c2 * (4 + vb),
                "flops": 2 * (f1 + f2)}
    if f == "batch":
        total = {"bytes": 0, "flops": 0}
        As, Bs = _batch(case["count"], case["n_hi"], 0, DTYPES[case["dtype"]])
        for A, B in zip(As, Bs):
            fm, nnz = _counts(A, B)
            total["bytes"] += _bytes(A) + _bytes(B) + 4 * (A.nrows + 1) + nnz * (vb + (0 if case["mode"] == "values" else 4))
            total["flops"] += 2 * fm
        return total
    A, B = _operands(case, 0)
    if f == "triangles":  # A, B and the mask are one matrix; half of the multiplications or more miss the mask
        fm, _ = _counts(A, B)
        return {"bytes": _bytes(A, not case["structural"]) + A.nnz * vb, "flops": 2 * fm}
    fm, nnz = _counts(A, B)
    inputs = _bytes(A) + (0 if A is B else _bytes(B))
    if f == "train":  # forward C; backward G and the operands again, two products per multiplication
        return {"bytes": 2 * inputs + nnz * (4 + vb) + nnz * (4 + vb) + (A.nnz + B.nnz) * vb, "flops": 6 * fm}
    rp = A.row_ptr.element_size() * (A.nrows + 1)
    return {"bytes": inputs + rp + nnz * (vb + (0 if case["mode"] == "values" else 4)), "flops": 2 * fm}


# ------------------------------------------------------------------ the same values from plain torch, FP64
CHUNK = 1 << 26  # products expanded at a time


def _chunks(A, B):
    """Products of A*B in blocks of A's rows: (first row, end row, entry of A, entry of B, row, column)."""
    arp, brp = A.row_ptr.long(), B.row_ptr.long()
    aci, bci = A.col_idx.long(), B.col_idx.long()
    blen = brp[1:] - brp[:-1]
    per = torch.zeros(A.nnz + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(blen[aci], 0, out=per[1:])
    row_end = per[arp]  # products before each row
    host = row_end.cpu()
    r0 = 0
    while r0 < A.nrows:
        r1 = int(torch.searchsorted(host, host[r0] + CHUNK, right=True)) - 1
        r1 = min(A.nrows, max(r1, r0 + 1))
        e0, e1 = int(arp[r0]), int(arp[r1])
        ent = torch.arange(e0, e1, device="cuda")
        cnt = blen[aci[e0:e1]]
        ea = torch.repeat_interleave(ent, cnt)
        eb = brp[aci[ea]] + torch.arange(ea.numel(), device="cuda") - (per[ea] - per[e0])
        row = torch.searchsorted(arp, ea, right=True) - 1
        yield r0, r1, ea, eb, row, bci[eb]
        r0 = r1


def _product(A, B):
    """(keys row * ncols + column of C's entries, values), in sorted order."""
    av, bv, keys, vals = A.values.double(), B.values.double(), [], []
    for _, _, ea, eb, row, col in _chunks(A, B):
        k, inv = torch.unique(row * B.ncols + col, return_inverse=True)
        vals.append(torch.zeros(k.numel(), dtype=torch.float64, device="cuda").index_add_(0, inv, av[ea] * bv[eb]))
        keys.append(k)
    return torch.cat(keys), torch.cat(vals)


def exact(case, seed):
    f, dtype = case["family"], DTYPES[case["dtype"]]
    if f == "galerkin":
        A = _stencil(27, case["g"], _gen(seed), dtype)
        P, Pt = _aggregation(case["g"], dtype)
        keys, vals = _product(A, P)
        AP = _csr(P.nrows, P.ncols, keys // P.ncols, keys % P.ncols, vals, torch.float64)
        # (the coarse product's exact values are those of exact A*P, also for FP32)
        return {"AP": {"row_ptr": None, "col_idx": None, "values": vals},
                "coarse": {"row_ptr": None, "col_idx": None, "values": _product(Pt, AP)[1]}}
    if f == "batch":
        As, Bs = _batch(case["count"], case["n_hi"], seed, dtype)
        return {"col_idx": None, "values": torch.cat([_product(A, B)[1] for A, B in zip(As, Bs)]),
                "row_ptr_first": None, "row_ptr_last": None}
    A, B = _operands(case, seed)
    if f == "triangles":
        rows = torch.repeat_interleave(torch.arange(A.nrows, device="cuda"), (A.row_ptr[1:] - A.row_ptr[:-1]).long())
        mask = rows * A.ncols + A.col_idx.long()
        out = torch.zeros(A.nnz, dtype=torch.float64, device="cuda")
        av = torch.ones_like(out) if case["structural"] else A.values.double()
        for _, _, ea, eb, row, col in _chunks(A, B):
            at = torch.searchsorted(mask, row * A.ncols + col).clamp_(max=mask.numel() - 1)
            hit = mask[at] == row * A.ncols + col
            out.index_add_(0, at[hit], av[ea[hit]] * av[eb[hit]])
        return out
    if f == "train":
        keys, vals = _product(A, B)
        gc = _normal(_gen(seed + 1000003), keys.numel()).to(dtype).double()
        av, bv, da, db = A.values.double(), B.values.double(), None, None
        da, db = torch.zeros_like(av), torch.zeros_like(bv)
        for _, _, ea, eb, row, col in _chunks(A, B):
            gp = gc[torch.searchsorted(keys, row * B.ncols + col)]
            da.index_add_(0, ea, gp * bv[eb])
            db.index_add_(0, eb, gp * av[ea])
        return {"c": vals, "da": da, "db": db}
    return {"row_ptr": None, "col_idx": None, "values": _product(A, B)[1]}
