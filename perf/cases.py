"""The work that users of this library have it do, as measurable cases.

Products y = alpha A x + beta y in every storage format and value type, Krylov
solves, mixed-precision refinement, the batched engine and PageRank, each
through the Python binding's public entry points, on the kinds of matrices
that the benchmark and the tests use: 5-, 7- and 27-point stencils, power-law
rows, random SPD matrices and upwind convection-diffusion, with values drawn
from the seed (heterogeneous coefficients, as a discretised problem has).

Linear systems are implicit steps (the operator plus a multiple of the
identity) solved to a tight tolerance, so that two correct solvers return the
same x to nine digits whatever the order of their additions.
"""
import functools
import math

import numpy as np
import torch

from paper_2103_10116_amd import inputs as I
from paper_2103_10116_amd import mxs

DEV = "cuda"
SHIFT = 0.1     # multiple of the identity in the systems that are solved
TOL = 1e-12
RESTART = 30
KMAX = 4096     # longest power-law row


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: one product of a small grid, where launch and
        # binding latency count
        dict(name="spmv_5pt_64_csr_f64", op="spmv", pattern="5pt", size=64, fmt="csr",
             dtype="f64", alpha=1.0, beta=0.0),
        # the benchmark's matrix: a large regular stencil in the default format ...
        dict(name="spmv_27pt_128_csr_f64", op="spmv", pattern="27pt", size=128, fmt="csr",
             dtype="f64", alpha=1.0, beta=0.0),
        # ... and in the format whose product moves the most bytes
        dict(name="spmv_27pt_128_coo_f64", op="spmv", pattern="27pt", size=128, fmt="coo",
             dtype="f64", alpha=1.0, beta=0.0),
        # single precision, padded format, an odd grid, y updated in place
        dict(name="spmv_27pt_101_ell_f32", op="spmv", pattern="27pt", size=101, fmt="ell",
             dtype="f32", alpha=0.75, beta=0.5),
        # circuit-like rows: power-law lengths, columns all over x
        dict(name="spmv_powerlaw_1048576_csr_f64", op="spmv", pattern="powerlaw", size=1048576,
             s=1.79, fmt="csr", dtype="f64", alpha=1.0, beta=0.0),
        dict(name="spmv_powerlaw_1000003_hyb_f32", op="spmv", pattern="powerlaw", size=1000003,
             s=2.0, fmt="hyb", dtype="f32", alpha=1.0, beta=1.0),
        # a small implicit step: the whole solve is latency
        dict(name="cg_5pt_64", op="solve", solver="cg", pattern="5pt", size=64),
        # a large implicit step by CG
        dict(name="cg_7pt_128", op="solve", solver="cg", pattern="7pt", size=128),
        # a nonsymmetric system by restarted GMRES
        dict(name="gmres_convdiff_100", op="solve", solver="gmres", pattern="convdiff", size=100),
        # an irregular SPD system by Jacobi-preconditioned CG
        dict(name="pcg_spd_1048576", op="solve", solver="pcg", pattern="spd", size=1048576, s=2.0),
        # mixed precision: FP64 refinement around CG on row-scaled FP16 values
        dict(name="ir_7pt_120_f16", op="ir", pattern="7pt", size=120, dtype="f16"),
        # serving: a burst of independent small systems through the batched engine
        dict(name="batch_256", op="batch", size=256),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["spmv", "solve", "ir", "batch", "pagerank"], [10, 6, 2, 1, 1])[0]
    if op == "spmv":
        pattern = rng.choice(["5pt", "7pt", "27pt", "powerlaw"])
        fmt = rng.choice(["csr", "csr", "coo", "ell", "hyb"])
        if pattern == "powerlaw" and fmt == "ell":
            fmt = "hyb"     # (padding every row to the longest one is not what a user does)
        dtype = rng.choice(["f64", "f64", "f32", "f32", "f16", "c128", "c64"]
                           if fmt == "csr" else ["f64", "f32"])
        c = dict(op=op, pattern=pattern, fmt=fmt, dtype=dtype,
                 alpha=rng.choice([1.0, -1.0, 0.75]), beta=rng.choice([0.0, 0.0, 1.0, 0.5]))
        c["size"] = {"5pt": lambda: _log(rng, 48, 1400), "7pt": lambda: _log(rng, 16, 128),
                     "27pt": lambda: _log(rng, 16, 100 if dtype == "c128" else 127),
                     "powerlaw": lambda: _log(rng, 1 << 14, 1 << 20)}[pattern]()
        if pattern == "powerlaw":
            c["s"] = rng.choice([1.79, 2.0])
        return c
    if op == "solve":
        solver = rng.choice(["cg", "pcg", "pipecg", "bicgstab", "cgs", "gmres"])
        pattern = {"cg": ["5pt", "7pt"], "pipecg": ["5pt", "7pt"],
                   "pcg": ["spd", "7pt"]}.get(solver, ["convdiff"])
        pattern = rng.choice(pattern)
        size = {"5pt": lambda: _log(rng, 40, 1000), "7pt": lambda: _log(rng, 14, 120),
                "convdiff": lambda: _log(rng, 14, 100),
                "spd": lambda: _log(rng, 1 << 13, 1 << 20)}[pattern]()
        c = dict(op=op, solver=solver, pattern=pattern, size=size)
        if pattern == "spd":
            c["s"] = 2.0
        return c
    if op == "ir":
        return dict(op=op, pattern="7pt", size=_log(rng, 24, 120),
                    dtype=rng.choice(["f16", "f32"]))
    if op == "batch":
        return dict(op=op, size=_log(rng, 16, 256))
    return dict(op=op, pattern="powerlaw", size=_log(rng, 1 << 14, 1 << 20), s=1.79)


# ---------------------------------------------------------------------------
# inputs, made on the GPU from the seed
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=1)
def _ctx():
    """The program's context, bound to torch's current stream."""
    return mxs.Context(torch.cuda.current_device())


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float64) * (hi - lo) + lo


def _csr(n, cols, vals, mask):
    """CSR of rows given as [n, k] tables whose columns ascend along k."""
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = mask.sum(1).cumsum(0)
    return n, rowptr.int(), cols[mask].int(), vals[mask]


def _grid(dims):
    """Coordinates (x fastest) and linear index of a grid's cells."""
    n = math.prod(dims)
    idx = torch.arange(n, device=DEV)
    coords, rest = [], idx
    for d in dims:
        coords.append(rest % d)
        rest = rest // d
    return n, idx, coords


def _stencil27(N, g):
    """27-point pattern, diagonal 26, the other coefficients -U[0.5, 1.5]."""
    n, idx, (x, y, z) = _grid((N, N, N))
    cols, mask = [], []
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                ok = torch.ones(n, dtype=torch.bool, device=DEV)
                for c, o in ((x, dx), (y, dy), (z, dz)):
                    if o:
                        ok &= (c + o >= 0) & (c + o < N)
                cols.append(idx + dx + dy * N + dz * N * N)
                mask.append(ok)
    vals = -_uniform(g, (n, 27), 0.5, 1.5)
    vals[:, 13] = 26.0
    return _csr(n, torch.stack(cols, 1), vals, torch.stack(mask, 1))


def _diffusion(dims, g, wind=0.0):
    """Weighted Dirichlet Laplacian (edge weights U[0.5, 1.5]) plus SHIFT on
    the diagonal; wind > 0 adds first-order upwind convection."""
    n, idx, coords = _grid(dims)
    lo, hi, strides = [], [], [math.prod(dims[:d]) for d in range(len(dims))]
    diag = torch.full((n,), SHIFT, dtype=torch.float64, device=DEV)
    for d, m in enumerate(dims):
        w = _uniform(g, (n,), 0.5, 1.5)              # edge to the next cell along d
        ghost = _uniform(g, (n,), 0.5, 1.5)          # boundary edge before the first cell
        before = torch.where(coords[d] > 0, torch.roll(w, strides[d]), ghost)
        conv = wind / (m + 1)
        diag += before + w + conv
        lo.append((idx - strides[d], -(before + conv), coords[d] > 0))
        hi.append((idx + strides[d], -w, coords[d] < m - 1))
    every = lo[::-1] + [(idx, diag, torch.ones(n, dtype=torch.bool, device=DEV))] + hi
    return _csr(n, *(torch.stack([e[k] for e in every], 1) for k in range(3)))


def _powerlaw_keys(n, s, g):
    """Sorted distinct keys row * n + col: Zipf(s) row lengths clipped to
    KMAX, columns uniform (a row's repeated columns count once)."""
    p = torch.arange(1, KMAX + 1, dtype=torch.float64, device=DEV) ** -s
    # (the mass beyond KMAX falls on KMAX, as clipping puts it)
    p[-1] += KMAX ** (1.0 - s) / (s - 1.0)
    cdf = torch.cumsum(p / p.sum(), 0)
    L = torch.searchsorted(cdf, _uniform(g, (n,), 0.0, 1.0)).clamp_(max=KMAX - 1) + 1
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), L)
    cols = torch.randint(0, n, rows.shape, generator=g, device=DEV)
    return torch.unique(rows * n + cols)


def _from_keys(n, key, val):
    rows = key // n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.bincount(rows, minlength=n).cumsum(0)
    return n, rowptr.int(), (key % n).int(), val


def _spd(n, s, g):
    """(P + P^T)/2 of the power-law pattern, diagonal 1.1 times the row's
    absolute sum (1 for an empty row): symmetric and diagonally dominant."""
    key = _powerlaw_keys(n, s, g)
    v = _uniform(g, key.shape, -0.5, 0.5)
    r, c = key // n, key % n
    off = r != c
    r, c, v = r[off], c[off], v[off]
    keys, inv = torch.unique(torch.cat([r * n + c, c * n + r]), return_inverse=True)
    # (an entry has at most two contributions, whose sum has one value in either order)
    sym = torch.zeros(keys.shape, dtype=torch.float64, device=DEV)
    sym.index_add_(0, inv, torch.cat([v, v]))
    _, rp, _, _ = _from_keys(n, keys, sym)
    cum = torch.zeros(keys.numel() + 1, dtype=torch.float64, device=DEV)
    cum[1:] = torch.round(sym.abs() * 2.0 ** 30).cumsum(0) * 2.0 ** -30  # exact sums
    absrow = cum[rp[1:].long()] - cum[rp[:-1].long()]
    d = torch.where(absrow > 0, 1.1 * absrow + 2.0 ** -16, torch.ones_like(absrow))
    ii = torch.arange(n, device=DEV)
    key, order = torch.sort(torch.cat([keys, ii * n + ii]))
    return _from_keys(n, key, torch.cat([sym, d])[order])


def _matrix(case, g):
    """(n, rowptr, col, val) on the GPU."""
    m, pat = case["size"], case["pattern"]
    if pat == "powerlaw":
        key = _powerlaw_keys(m, case["s"], g)
        return _from_keys(m, key, _uniform(g, key.shape, -1.0, 1.0))
    if pat == "spd":
        return _spd(m, case["s"], g)
    if pat == "27pt":
        return _stencil27(m, g)
    if pat == "convdiff":
        return _diffusion((m, m, m), g, wind=10.0)
    return _diffusion((m,) * (2 if pat == "5pt" else 3), g)


_VEC = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float32,
        "c128": torch.complex128, "c64": torch.complex64}


def _spmv_inputs(case, seed):
    """The matrix (complex values as a complex tensor), x and the old y."""
    g = _gen(seed)
    n, rp, ci, v = _matrix(case, g)
    cplx = case["dtype"] in ("c128", "c64")
    if cplx:
        v = torch.complex(v, _uniform(g, v.shape, -1.0, 1.0))
    parts = [_uniform(g, (n,), -1.0, 1.0) for _ in range(4 if cplx else 2)]
    x, y = (torch.complex(*parts[:2]), torch.complex(*parts[2:])) if cplx else parts
    dt = _VEC[case["dtype"]]
    return n, rp, ci, v, x.to(dt), y.to(dt)


def _system_inputs(case, seed):
    g = _gen(seed)
    n, rp, ci, v = _matrix(case, g)
    return n, rp, ci, v, _uniform(g, (n,), -1.0, 1.0)


def _batch_inputs(case, seed):
    """Serving requests: grid sides of the benchmark's request stream, weights
    and right-hand sides from the seed."""
    r = np.random.Generator(np.random.Philox(int(seed)))
    out = []
    for q in I.serving_stream(case["size"], 0.0):
        sd = int(r.integers(1, 2**31 - 1))
        A = I.serving_system(q.m, sd)
        out.append((A, I.serving_rhs(A.n, sd)))
    return out


def _graph_inputs(case, seed):
    """In-link pattern of a directed graph (power-law in-degrees), host arrays."""
    g = _gen(seed)
    n, rp, ci, _ = _from_keys(case["size"], *(2 * [_powerlaw_keys(case["size"], case["s"], g)]))
    return I.CSRMatrix(n, n, rp.cpu().numpy(), ci.cpu().numpy(), None)


# ---------------------------------------------------------------------------
# what a program holds before the call, and the call
# ---------------------------------------------------------------------------
def prepare(case, seed):
    ctx, op = _ctx(), case["op"]
    st = dict(case=case, ctx=ctx)
    if op == "spmv":
        n, rp, ci, v, x, y = _spmv_inputs(case, seed)
        if v.is_complex():
            M = mxs.Matrix.from_host_complex(ctx, n, n, rp.cpu().numpy(), ci.cpu().numpy(),
                                             v.cpu().numpy())
        else:
            M = mxs.Matrix.from_csr(ctx, n, n, rp, ci, v)
        home = ("csr", "c128") if v.is_complex() else ("csr", "f64")
        if (case["fmt"], case["dtype"]) != home:
            M = M.convert(case["fmt"], case["dtype"])
        st.update(A=M, x=x, y0=y, y=y.clone())
    elif op in ("solve", "ir"):
        n, rp, ci, v, b = _system_inputs(case, seed)
        st.update(A=mxs.Matrix.from_csr(ctx, n, n, rp, ci, v), b=b)
        if op == "ir":
            st["low"] = st["A"].convert("csr", case["dtype"])
        elif case["solver"] == "pcg":
            st["precond"] = mxs.Precond(ctx, st["A"], "jacobi")
    elif op == "batch":
        st["systems"] = _batch_inputs(case, seed)
        st["engine"] = mxs.Batch(ctx, budget_bytes=256 << 20, max_slots=1024)
    else:
        st["graph"] = mxs.Graph(ctx, _graph_inputs(case, seed))
        st["x"] = torch.empty(case["size"], dtype=torch.float64, device=DEV)
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    op = case["op"]
    if op == "spmv":
        if case["beta"]:
            st["y"].copy_(st["y0"])      # the y that the product updates
        mxs.spmv(ctx, st["A"], st["x"], st["y"], case["alpha"], case["beta"])
        return st["y"]
    if op == "solve":
        x = torch.zeros_like(st["b"])
        kind = "cg" if case["solver"] == "pcg" else case["solver"]
        mxs.solve(ctx, kind, st["A"], st["b"], x, tol=TOL, restart=RESTART,
                  precond=st.get("precond"))
        return x
    if op == "ir":
        x = torch.zeros_like(st["b"])
        mxs.solve_ir(ctx, st["A"], st["low"], st["b"], x, tol=TOL, carry_direction=True)
        return x
    if op == "batch":
        B, systems = st["engine"], st["systems"]
        tickets, _ = B.submit_many(systems, tol=TOL)
        left = len(systems)
        while left:
            B.step()
            left -= len(B.completed())
        statuses, x, _, _ = B.poll_many(tickets, [A.n for A, _ in systems])
        return x, statuses
    mxs.pagerank(ctx, st["graph"], st["x"], tol=1e-12)
    return st["x"]


# ---------------------------------------------------------------------------
# what one pass cannot do without
# ---------------------------------------------------------------------------
def _mean_row(s):
    k = np.arange(1, KMAX + 1, dtype=np.float64)
    p = k ** -s
    p[-1] += KMAX ** (1.0 - s) / (s - 1.0)
    return float((k * p).sum() / p.sum())


def _shape(case):
    """(n, entries) of the case's matrix."""
    m = case["size"]
    if case["pattern"] == "5pt":
        return m * m, 5 * m * m - 4 * m
    if case["pattern"] in ("7pt", "convdiff"):
        return m ** 3, 7 * m ** 3 - 6 * m * m
    if case["pattern"] == "27pt":
        return m ** 3, (3 * m - 2) ** 3
    nnz = m * _mean_row(case["s"])
    return m, nnz if case["pattern"] == "powerlaw" else 2 * nnz + m


def work(case):
    op = case["op"]
    if op == "batch":
        # systems of 2700 rows on average: read once, b read and x written once
        n = 2700.0 * case["size"]
        return {"bytes": n * (5 * 12 + 4 + 16), "flops": n * 100 * 20}
    n, nnz = _shape(case)
    if op == "spmv":
        vb = {"f64": 8, "f32": 4, "f16": 2, "c128": 16, "c64": 8}[case["dtype"]]
        xb = {"f16": 4}.get(case["dtype"], vb)
        idx = 8 if case["fmt"] == "coo" else 4
        rows = 4 * (n + 1) if case["fmt"] == "csr" else 0
        flops = 8 if case["dtype"][0] == "c" else 2
        return {"bytes": nnz * (vb + idx) + rows + (2 + (case["beta"] != 0)) * n * xb,
                "flops": flops * nnz}
    csr = 12 * nnz + 4 * (n + 1)
    if op == "pagerank":
        return {"bytes": 20 * (csr + 25 * n), "flops": 20 * (2 * nnz + 5 * n)}
    # iterations from the condition number's bound on CG's convergence
    kappa = {"5pt": 16, "7pt": 24, "convdiff": 24}.get(case["pattern"], 2.1 * SHIFT) / SHIFT
    its = 0.35 * math.sqrt(kappa) * math.log(2 / TOL)
    if op == "ir":
        low = (4 + (2 if case["dtype"] == "f16" else 4)) * nnz + 8 * n
        return {"bytes": its * (low + 32 * n), "flops": its * (2 * nnz + 10 * n)}
    per = {"cg": (1, 8), "pcg": (1, 10), "pipecg": (1, 13), "bicgstab": (2, 15), "cgs": (2, 16),
           "gmres": (1, 2.0 * RESTART / 2 + 6)}[case["solver"]]
    if per[0] == 2:
        its /= 2
    return {"bytes": its * (per[0] * csr + per[1] * 8 * n),
            "flops": its * (per[0] * 2 * nnz + per[1] * n)}


# ---------------------------------------------------------------------------
# the same in 64 bits by plain torch
# ---------------------------------------------------------------------------
def _sparse(n, rp, ci, v):
    return torch.sparse_csr_tensor(rp.long(), ci.long(), v, size=(n, n))


def _refine(A, b, diag, symmetric):
    """Solves A x = b until the residual stops falling: refinement steps around
    Jacobi-preconditioned CG, or BiCGSTAB for a nonsymmetric A."""
    inner = _pcg if symmetric else _bicgstab
    x = torch.zeros_like(b)
    best, at = math.inf, x
    for _ in range(8):
        r = b - A @ x
        rn = float(r.norm())
        if rn < best:
            at = x
        if rn >= 0.5 * best:
            break
        best = rn
        x = x + inner(A, r, diag)
    return at


def _pcg(A, b, diag, tol=1e-7):
    x, r = torch.zeros_like(b), b.clone()
    p = r / diag
    rz, target = torch.dot(r, p), tol * float(b.norm())
    for k in range(3000):
        q = A @ p
        a = rz / torch.dot(p, q)
        x += a * p
        r -= a * q
        if k % 10 == 9 and float(r.norm()) <= target:
            break
        z = r / diag
        new = torch.dot(r, z)
        p = z + (new / rz) * p
        rz = new
    return x


def _bicgstab(A, b, diag, tol=1e-7):
    x, r = torch.zeros_like(b), b.clone()
    rh, p, target = r.clone(), r.clone(), tol * float(b.norm())
    rho = torch.dot(rh, r)
    for _ in range(3000):
        v = A @ p
        a = rho / torch.dot(rh, v)
        s = r - a * v
        t = A @ s
        w = torch.dot(t, s) / torch.dot(t, t)
        x += a * p + w * s
        r = s - w * t
        if float(r.norm()) <= target:
            break
        new = torch.dot(rh, r)
        p = r + (new / rho) * (a / w) * (p - w * v)
        rho = new
    return x


def exact(case, seed):
    op = case["op"]
    if op == "spmv":
        n, rp, ci, v, x, y = _spmv_inputs(case, seed)
        dt = case["dtype"]
        wide = torch.complex128 if v.is_complex() else torch.float64
        rows = torch.repeat_interleave(torch.arange(n, device=DEV), rp.diff().long())
        if dt == "f32":
            v = v.float()
        elif dt == "c64":
            v = v.to(torch.complex64)
        elif dt == "f16":
            # half-precision values scaled by a power of two per row
            top = torch.zeros(n, dtype=torch.float64, device=DEV)
            top.scatter_reduce_(0, rows, v.abs(), "amax")
            sc = torch.exp2(torch.ceil(torch.log2(top)))[rows]
            v = (v / sc).half().double() * sc
        prod = v.to(wide) * x.to(wide)[ci.long()]
        out = torch.zeros(n, dtype=wide, device=DEV)
        if wide == torch.complex128:
            for part in (torch.real, torch.imag):
                part(out).index_add_(0, rows, part(prod))
        else:
            out.index_add_(0, rows, prod)
        return case["alpha"] * out + case["beta"] * y.to(wide)
    if op in ("solve", "ir"):
        n, rp, ci, v, b = _system_inputs(case, seed)
        rows = torch.repeat_interleave(torch.arange(n, device=DEV), rp.diff().long())
        diag = v[rows == ci.long()]
        return _refine(_sparse(n, rp, ci, v), b, diag, case["pattern"] != "convdiff")
    if op == "batch":
        systems = _batch_inputs(case, seed)
        cols, ptrs, base, nnz = [], [np.zeros(1, np.int64)], 0, 0
        for A, _ in systems:
            cols.append(A.col.astype(np.int64) + base)
            ptrs.append(A.rowptr[1:].astype(np.int64) + nnz)
            base += A.n
            nnz += A.nnz
        rp, ci, v, b = (torch.from_numpy(np.concatenate(a)).to(DEV) for a in
                        (ptrs, cols, [A.val for A, _ in systems], [q for _, q in systems]))
        rows = torch.repeat_interleave(torch.arange(base, device=DEV), rp.diff())
        return _refine(_sparse(base, rp, ci, v), b, v[rows == ci], True), None
    G = _graph_inputs(case, seed)
    n = G.n
    rp, ci = (torch.from_numpy(a.astype(np.int64)).to(DEV) for a in (G.rowptr, G.col))
    deg = torch.bincount(ci, minlength=n).double()
    A = _sparse(n, rp, ci, 1.0 / deg[ci])
    x = torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
    for _ in range(200):
        new = 0.85 * (A @ x + x[deg == 0].sum() / n) + 0.15 / n
        change = float((new - x).abs().sum())
        x = new
        if change <= 1e-15:
            break
    return x
