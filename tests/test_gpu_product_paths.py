"""Which product a matrix takes where two rules meet, and the products inside
solvers that no other test reaches: the two passes near their largest number of
column panels, the FP32 and row-scaled FP16 dot products of both new forms in
refinement's inner solves, preconditioned CG's p.q from the bins, and more bins
than dot partials."""
import numpy as np
import pytest

from paper_2103_10116_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2103_10116_amd import mxs
    ctx = mxs.Context(0)
    yield mxs, ctx, torch
    ctx.close()


def _shared_columns(ncols, lens, seed):
    """Rows of the given lengths, one column drawn from each equal share."""
    g = I.rng(seed)
    lens = np.asarray(lens, np.int64)
    rp = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    rows = np.repeat(np.arange(len(lens)), lens)
    L = lens[rows]
    j = np.arange(rp[-1]) - rp[rows]
    lo, hi = j * ncols // L, (j + 1) * ncols // L
    col = lo + (g.random(len(lo)) * (hi - lo)).astype(np.int64)
    return I.CSRMatrix(len(lens), ncols, rp.astype(np.int32), col.astype(np.int32),
                       g.uniform(-1, 1, len(col)))


# columns on either side of 128 panels (20448 FP64 or 32768 FP32 columns each),
# at 147 of them and on either side of 160, the most that the two passes take
PANELS = [("f64", 128 * 20448, True), ("f64", 128 * 20448 + 1, True), ("f64", 3000001, True),
          ("f64", 160 * 20448, True), ("f64", 160 * 20448 + 1, False),
          ("f32", 128 * 32768 + 1, True), ("f32", 160 * 32768, True),
          ("f32", 160 * 32768 + 1, False), ("f16", 4800001, True)]


@pytest.mark.parametrize("dt,ncols,takes", PANELS)
def test_most_panels(env, orc, dt, ncols, takes):
    """The path itself: a matrix whose kernel is asked for keeps the arrays of
    the column panels, so AUTO's bytes are the same exactly when it falls back
    on them."""
    mxs, ctx, torch = env
    A = _shared_columns(ncols, [30] * 20000 + [100], 11)
    M = mxs.Matrix.from_host(ctx, A)
    B, P = M.convert("csr", dt), M.convert("csr", dt, csr_kernel="merge")
    assert (B.info()["bytes"] != P.info()["bytes"]) == takes
    x, y0, val = I.uniform_vector(ncols, 12), I.uniform_vector(A.n, 13), A.val
    if dt != "f64":
        x, y0, val = (v.astype(np.float32).astype(np.float64) for v in (x, y0, val))
    if dt == "f16":
        _, h, s = orc.rowscale_f16(A)
        val = orc.f16_bits_to_f64(h) * np.repeat(s.astype(np.float64), A.row_lengths())
    R = I.CSRMatrix(A.n, ncols, A.rowptr, A.col, val)
    tdt = torch.float64 if dt == "f64" else torch.float32
    ya = torch.from_numpy(y0).to(tdt).cuda()
    yb = ya.clone()
    xd = torch.from_numpy(x).to(tdt).cuda()
    mxs.spmv(ctx, B, xd, ya, 1.5, -0.5)
    mxs.spmv(ctx, B, xd, yb, 1.5, -0.5, noalloc=True)
    err = np.abs(ya.cpu().numpy().astype(np.float64) - orc.spmv_csr(R, x, 1.5, -0.5, y0))
    tol = 1e-13 if dt == "f64" else 1e-5
    assert (err <= tol * (1.5 * orc.absrow(R, x) + 0.5 * np.abs(y0)) + 1e-30).all()
    assert torch.equal(ya, yb)
    for m in (B, P, M):
        m.close()


def _slack(orc, A, b, x):
    """Rounding of the residual's own evaluation."""
    return 64 * 2.0 ** -53 * np.linalg.norm(np.abs(b) + orc.absrow(A, x)) / np.linalg.norm(b)


def _spd():
    A = I.random_spd(1 << 16, seed=31)
    rows = np.repeat(np.arange(A.n), A.row_lengths())
    A.val[rows == A.col] *= 4.0
    return A


@pytest.mark.parametrize("carry", [False, True])
@pytest.mark.parametrize("precond", [None, "jacobi", "block_jacobi"])
@pytest.mark.parametrize("low", ["f32", "f16"])
@pytest.mark.parametrize("system", ["grid", "powerlaw"])
def test_refinement_inner_products(env, orc, system, low, precond, carry):
    """The inner CG's p.q from FP32 and row-scaled FP16 products over diagonals
    (31^3: a last work-group and slice that are not full) and over bins."""
    mxs, ctx, torch = env
    A = I.poisson3d(31) if system == "grid" else _spd()
    b = I.uniform_vector(A.n, 61)
    M = mxs.Matrix.from_host(ctx, A)
    L = M.convert("csr", low)
    kept = M.convert("csr", low, csr_kernel="rows_lds" if system == "grid" else "merge")
    assert L.info()["bytes"] > kept.info()["bytes"]        # the second copy
    P = mxs.Precond(ctx, M, precond, 4) if precond else None
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    r = mxs.solve_ir(ctx, M, L, torch.from_numpy(b).cuda(), x, tol=1e-10, precond=P,
                     carry_direction=carry)
    xh = x.cpu().numpy()
    assert r.status == mxs.OK
    assert orc.true_relres(A, b, xh) <= 1e-10 + _slack(orc, A, b, xh)
    # the same steps as with the products that form no dots of this kind
    x2 = torch.zeros_like(x)
    r2 = mxs.solve_ir(ctx, M, kept, torch.from_numpy(b).cuda(), x2, tol=1e-10, precond=P,
                      carry_direction=carry)
    assert abs(r.outer_iters - r2.outer_iters) <= 1
    assert abs(r.inner_iters_total - r2.inner_iters_total) <= 0.1 * r2.inner_iters_total + 2


@pytest.mark.parametrize("kind,bs", [("jacobi", 1), ("block_jacobi", 8)])
@pytest.mark.parametrize("system", ["grid", "powerlaw"])
def test_preconditioned_cg_products(env, orc, system, kind, bs):
    mxs, ctx, torch = env
    A = I.poisson3d(31) if system == "grid" else _spd()
    b = I.uniform_vector(A.n, 62)
    M = mxs.Matrix.from_host(ctx, A)
    P = mxs.Precond(ctx, M, kind, bs)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    r = mxs.solve(ctx, "cg", M, torch.from_numpy(b).cuda(), x, tol=1e-10, precond=P)
    xh = x.cpu().numpy()
    assert orc.true_relres(A, b, xh) <= 1e-10 + _slack(orc, A, b, xh)
    ref = orc.pcg(A, b, orc.jacobi(A)[1] if kind == "jacobi" else orc.block_jacobi(A, bs)[1],
                  tol=1e-10)
    assert abs(r.iters - ref.iters) <= max(3, ref.iters // 10)


@pytest.mark.parametrize("solver", ["cg", "bicgstab"])
def test_more_bins_than_dot_partials(env, orc, solver):
    """2^21 rows whose 11 entries lie in 11 panels, so that a bin of 4096
    partial sums holds 372 rows: 5600 bins, beyond the 4096 dot partials; the
    solvers form their dots apart from the product."""
    mxs, ctx, torch = env
    n = 1 << 21
    g = I.rng(71)
    # circulant edges at five distances, and row 0 joined to 100 others
    far = (np.array([1, 2, 3, 4, 5]) * (n // 11) + g.integers(0, 1000, 5)).astype(np.int64)
    i = np.arange(n, dtype=np.int64)
    rows = np.concatenate([np.tile(i, 5), np.zeros(100, np.int64)])
    cols = np.concatenate([(i + d) % n for d in far] + [np.arange(1, 101) * 20001])
    assert not np.isin(cols[-100:], np.concatenate([far, (n - far) % n])).any()
    w = g.uniform(-1, 1, len(rows))
    r, c = np.concatenate([rows, cols, i]), np.concatenate([cols, rows, i])
    v = np.concatenate([w, w, np.where(i == 0, 150.0, 14.0)])
    order = np.lexsort((c, r))
    r, c, v = r[order], c[order], v[order]
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(r, minlength=n), out=rp[1:])
    A = I.CSRMatrix(n, n, rp.astype(np.int32), c.astype(np.int32), v)
    assert A.row_lengths().max() > 64
    M = mxs.Matrix.from_host(ctx, A)
    P = M.convert("csr", "f64", csr_kernel="merge")
    assert M.info()["bytes"] != P.info()["bytes"]          # the two passes
    P.close()
    b = I.uniform_vector(n, 72)
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    mxs.solve(ctx, solver, M, torch.from_numpy(b).cuda(), x, tol=1e-10)
    xh = x.cpu().numpy()
    assert orc.true_relres(A, b, xh) <= 1e-10 + _slack(orc, A, b, xh)
    M.close()


def _band(n, per, half, seed):
    """Rows of `per` entries, one in each equal share of the 2 half + 1 columns
    about the diagonal."""
    g = I.rng(seed)
    share = (2 * half + 1) // per
    base = np.clip(np.arange(n) - half, 0, n - 2 * half - 1)
    col = base[:, None] + np.arange(per) * share + g.integers(0, share, (n, per))
    return I.CSRMatrix(n, n, np.arange(0, n * per + 1, per, dtype=np.int32),
                       col.reshape(-1).astype(np.int32), g.uniform(-1, 1, n * per))


def _unknowns3(N):
    """Three unknowns at each node of a 27-point grid (rows of 81)."""
    P = I.stencil27(N)
    lens = np.repeat(P.row_lengths() * 3, 3)
    rp = np.zeros(3 * P.n + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    cols = (P.col[:, None].astype(np.int64) * 3 + np.arange(3)).ravel()
    node = np.repeat(np.arange(P.n), 3)
    off = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    col = cols[np.repeat(P.rowptr[:-1].astype(np.int64)[node] * 3, lens) + off]
    v = np.where(col == np.repeat(np.arange(3 * P.n), lens), 90.0, -1.0)
    return I.CSRMatrix(3 * P.n, 3 * P.n, rp.astype(np.int32), col.astype(np.int32), v)


@pytest.mark.parametrize("name,near", [("band_200", True), ("band_600", True),
                                       ("band_2000", False), ("grid", True), ("scattered", False)])
def test_rows_whose_columns_are_near(env, orc, name, near):
    """FP64 products of rows that share their columns stay on the merge path:
    they are its bits (chunks of 512 entries), where two passes add a row's
    products in runs of 8; FP32 ones run in two passes either way."""
    mxs, ctx, torch = env
    A = (_unknowns3(23) if name == "grid" else _spd() if name == "scattered"
         else _band(40000, 80, int(name[5:]), 81))
    A.val[:] = I.rng(82).uniform(-1, 1, A.nnz)
    M = mxs.Matrix.from_host(ctx, A)
    for dt in ("f64", "f32"):
        tdt = torch.float64 if dt == "f64" else torch.float32
        x = I.uniform_vector(A.n, 83)
        val = A.val
        if dt == "f32":
            x, val = (v.astype(np.float32).astype(np.float64) for v in (x, val))
        R = I.CSRMatrix(A.n, A.n, A.rowptr, A.col, val)
        xd = torch.from_numpy(x).to(tdt).cuda()
        ys = []
        for opts in ({}, dict(csr_kernel="merge")):
            B = M.convert("csr", dt, **opts)
            y, z = (torch.full((A.n,), float("nan"), dtype=tdt, device="cuda") for _ in range(2))
            mxs.spmv(ctx, B, xd, y)
            mxs.spmv(ctx, B, xd, z, noalloc=True)
            assert torch.equal(y, z)
            ys.append(y)
            B.close()
        err = np.abs(ys[0].cpu().numpy().astype(np.float64) - orc.spmv_csr(R, x))
        assert (err <= (1e-13 if dt == "f64" else 1e-5) * orc.absrow(R, x) + 1e-30).all()
        assert torch.equal(*ys) == (near and dt == "f64")
    M.close()


@pytest.mark.parametrize("kind", ["cg", "pcg", "bicgstab", "cgs", "gmres", "pipecg"])
def test_solvers_on_near_rows(env, orc, kind):
    """A solver's products (with and without dots) in two passes, a product by
    itself on the merge path, with the context's scratch growing in between."""
    mxs, _, torch = env
    ctx = mxs.Context(0)
    A = _unknowns3(23)
    b = I.uniform_vector(A.n, 84)
    M = mxs.Matrix.from_host(ctx, A)
    P = mxs.Precond(ctx, M, "jacobi") if kind == "pcg" else None
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    y = torch.zeros_like(x)
    mxs.spmv(ctx, M, torch.from_numpy(b).cuda(), y)
    err = np.abs(y.cpu().numpy() - orc.spmv_csr(A, b))
    assert (err <= 1e-13 * orc.absrow(A, b)).all()
    mxs.solve(ctx, "cg" if P else kind, M, torch.from_numpy(b).cuda(), x, tol=1e-10, precond=P)
    xh = x.cpu().numpy()
    assert orc.true_relres(A, b, xh) <= 1e-10 + _slack(orc, A, b, xh)
    if P:
        P.close()
    M.close()
    ctx.close()


def _diagonals(n, D, seed):
    """D diagonals, ten apart (no threes), all entries inside the matrix."""
    c = np.arange(n)[:, None] + (np.arange(D) - D // 2) * 10
    on = (c >= 0) & (c < n)
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(on.sum(1), out=rp[1:])
    return I.CSRMatrix(n, n, rp.astype(np.int32), c[on].astype(np.int32),
                       I.rng(seed).uniform(-1, 1, int(rp[-1])))


# rows on either side of each line: rounds of 9, 7, 5 or 8 diagonals times 6500
# (CSR FP64), 12000 (CSR FP32, FP16) or, from 6 rounds on, 4500 (COO); ELL by the
# diagonals (three terms add up alike in both kernels: their rows pin the values)
ROUNDS = [("csr", "f64", 27, 19499, False), ("csr", "f64", 27, 19500, True),
          ("csr", "f64", 64, 51999, False), ("csr", "f64", 64, 52000, True),
          ("csr", "f64", 9, 16000, True), ("csr", "f32", 13, 23999, False),
          ("csr", "f32", 13, 24000, True), ("csr", "f16", 27, 35999, False),
          ("csr", "f16", 27, 36000, True), ("coo", "f64", 48, 26999, False),
          ("coo", "f64", 48, 27000, True), ("coo", "f32", 64, 35999, False),
          ("coo", "f32", 64, 36000, True), ("coo", "f64", 32, 5000, True),
          ("ell", "f64", 3, 60000, False), ("ell", "f32", 4, 50000, True),
          ("hyb", "f64", 3, 60000, False), ("hyb", "f64", 4, 50000, True)]


@pytest.mark.parametrize("fmt,dt,D,n,over", ROUNDS)
def test_diagonals_of_few_rows(env, orc, fmt, dt, D, n, over):
    """Where the rows are few for their diagonals the format's own kernel runs:
    its bits, which the order of the sums over diagonals does not give."""
    mxs, ctx, torch = env
    A = _diagonals(n, D, 91)
    assert A.nnz >= 1 << 17
    M = mxs.Matrix.from_host(ctx, A)
    opts = {"csr": dict(csr_kernel="rows_lds" if D <= 8 or dt != "f64" else "products"),
            "coo": dict(coo_kernel="lds")}.get(fmt, dict(waves_per_group=4))
    x, val = I.uniform_vector(n, 92), A.val
    if dt != "f64":
        x, val = (v.astype(np.float32).astype(np.float64) for v in (x, val))
    if dt == "f16":
        _, h, s = orc.rowscale_f16(A)
        val = orc.f16_bits_to_f64(h) * np.repeat(s.astype(np.float64), A.row_lengths())
    R = I.CSRMatrix(n, n, A.rowptr, A.col, val)
    tdt = torch.float64 if dt == "f64" else torch.float32
    xd = torch.from_numpy(x).to(tdt).cuda()
    ys, kept = [], []
    for o in ({}, opts):
        B = M.convert(fmt, dt, **o)
        y, z = (torch.full((n,), float("nan"), dtype=tdt, device="cuda") for _ in range(2))
        mxs.spmv(ctx, B, xd, y)
        mxs.spmv(ctx, B, xd, z, noalloc=True)
        assert torch.equal(y, z)
        ys.append(y)
        kept.append(B.info()["bytes"])
        B.close()
    assert kept[0] > kept[1]                               # the copy by diagonals
    err = np.abs(ys[0].cpu().numpy().astype(np.float64) - orc.spmv_csr(R, x))
    assert (err <= (1e-13 if dt == "f64" else 1e-5) * orc.absrow(R, x) + 1e-30).all()
    assert torch.equal(*ys) == (not over)
    M.close()


@pytest.mark.parametrize("D,n", [(64, 4000), (64, 31000), (32, 10001), (27, 6000)])
@pytest.mark.parametrize("kind", ["cg", "pcg", "bicgstab", "cgs", "gmres", "pipecg"])
def test_solvers_on_diagonals_of_few_rows(env, orc, kind, D, n):
    """Products with dots over diagonals and plain ones by the format's kernel,
    and both by the latter (rows below the lines of both)."""
    mxs, ctx, torch = env
    A = _diagonals(n, D, 93)
    # symmetric: entry (i, j) and (j, i) by the same function of i + j
    rows = np.repeat(np.arange(n), A.row_lengths())
    A.val[:] = np.where(rows == A.col, 2.0 * D, -np.abs(np.sin(rows + A.col.astype(np.float64))))
    if D % 2 == 0:                                         # one diagonal without a mirror
        A.val[A.col == rows - D // 2 * 10] = 0.0
    b = I.uniform_vector(n, 94)
    M = mxs.Matrix.from_host(ctx, A)
    P = mxs.Precond(ctx, M, "jacobi") if kind == "pcg" else None
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    mxs.solve(ctx, "cg" if P else kind, M, torch.from_numpy(b).cuda(), x, tol=1e-10, precond=P)
    xh = x.cpu().numpy()
    assert orc.true_relres(A, b, xh) <= 1e-10 + _slack(orc, A, b, xh)
    if P:
        P.close()
    M.close()
