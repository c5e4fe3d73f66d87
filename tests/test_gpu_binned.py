"""The two-pass product of irregular matrices (row bins and column panels)
against the CPU oracle at the sizes where its layout can go wrong: the
smallest matrix that takes it, bins full of one-entry rows, rows longer than a
bin's lanes, many panels, several batches of bins; its dot products inside
the solvers and its values refreshed in place.

Chains of additions: at most 8 products a run, 8 partial sums a lane, a scan
of 6 steps and 8 waves, so at most 30 roundings: 3.4e-15 of sum |a||x| in
FP64, 1.8e-6 in FP32, within the library's 1e-13 and 1e-5."""
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


def _matrix(ncols, lens, seed):
    """Rows of the given lengths, one column drawn from each equal share of
    the columns (sorted and distinct)."""
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


def _lens(name):
    if name == "smallest":      # 32768 columns, 2^19 entries and a remainder
        return 32768, [65] * 8065 + [0, 0, 63] + [1]
    if name == "below":         # one entry fewer than the rule asks for
        return 32768, [65] * 8065 + [62]
    if name == "one_entry":     # bins limited by their rows; every third row empty
        return 40000, [1, 1, 0] * 300000 + [70]
    if name == "long":          # rows over many waves, and a row of 32000 entries
        return 300007, [32000] + [20000] * 20 + [3] * 40000 + [0] * 3000
    if name == "wide":          # 147 panels
        return 3000001, [30] * 20000 + [100]
    raise KeyError(name)


@pytest.mark.parametrize("name", ["smallest", "below", "one_entry", "long", "wide"])
def test_products(env, orc, name):
    mxs, ctx, torch = env
    ncols, lens = _lens(name)
    A = _matrix(ncols, lens, 11)
    assert (A.nnz < 1 << 19) == (name == "below")
    M = mxs.Matrix.from_host(ctx, A)
    x, y0 = I.uniform_vector(ncols, 12), I.uniform_vector(A.n, 13)
    for fmt, dt in (("csr", "f64"), ("csr", "f32"), ("csr", "f16"), ("coo", "f64"),
                    ("coo", "f32"), ("hyb", "f64"), ("hyb", "f32")):
        B = M.convert(fmt, dt)
        kept = B.info()["bytes"] / A.nnz   # the second copy of the entries
        vb = {"f64": 8, "f32": 4, "f16": 2}[dt]
        if fmt == "csr":
            assert (kept > 1.6 * (vb + 4)) == (name != "below"), (fmt, dt, kept)
        tdt = torch.float64 if dt == "f64" else torch.float32
        val, xr, yr = A.val, x, y0
        if dt != "f64":
            xr, yr = (v.astype(np.float32).astype(np.float64) for v in (x, y0))
            val = orc.cast_f32(A.val)[1].astype(np.float64)
        if dt == "f16":
            _, h, s = orc.rowscale_f16(A)
            val = orc.f16_bits_to_f64(h) * np.repeat(s.astype(np.float64), A.row_lengths())
        R = I.CSRMatrix(A.n, ncols, A.rowptr, A.col, val)
        tol = 1e-13 if dt == "f64" else 1e-5
        xd = torch.from_numpy(xr).to(tdt).cuda()
        y = torch.from_numpy(yr).to(tdt).cuda()
        mxs.spmv(ctx, B, xd, y, 1.5, -0.5)
        ref, scale = orc.spmv_csr(R, xr, 1.5, -0.5, yr), orc.absrow(R, xr)
        err = np.abs(y.cpu().numpy().astype(np.float64) - ref)
        assert (err <= tol * (1.5 * scale + 0.5 * np.abs(yr)) + 1e-30).all(), (fmt, dt)
        # beta = 0 never reads y; the allocation-free product is the same bits
        ya, yb = (torch.full((A.n,), float("nan"), dtype=tdt, device="cuda") for _ in range(2))
        mxs.spmv(ctx, B, xd, ya)
        mxs.spmv(ctx, B, xd, yb, noalloc=True)
        err = np.abs(ya.cpu().numpy().astype(np.float64) - orc.spmv_csr(R, xr))
        assert (err <= tol * scale + 1e-30).all() and torch.equal(ya, yb), (fmt, dt)
        B.close()


def test_batches(env, orc):
    """73 MB of FP64 partial sums: the allocation-free product takes the bins
    in two batches, with the same result; values that are not finite stay in
    their rows."""
    mxs, ctx, torch = env
    n = 1 << 20
    A = _matrix(n, [9] * n + [70], 21)
    B = mxs.Matrix.from_host(ctx, A)
    x = I.uniform_vector(n, 22)
    xd = torch.from_numpy(x).cuda()
    ya, yb = (torch.zeros(A.n, dtype=torch.float64, device="cuda") for _ in range(2))
    mxs.spmv(ctx, B, xd, ya)
    mxs.spmv(ctx, B, xd, yb, noalloc=True)
    assert torch.equal(ya, yb)
    err = np.abs(ya.cpu().numpy() - orc.spmv_csr(A, x))
    assert (err <= 1e-13 * orc.absrow(A, x)).all()
    c = int(A.col[12345])
    xd[c], xd[0] = float("inf"), float("nan")
    mxs.spmv(ctx, B, xd, ya)
    hit = np.unique(np.repeat(np.arange(A.n), A.row_lengths())[(A.col == c) | (A.col == 0)])
    bad = np.flatnonzero(~np.isfinite(ya.cpu().numpy()))
    assert np.array_equal(bad, hit)


@pytest.mark.parametrize("solver", ["cg", "bicgstab", "cgs"])
def test_dots_inside_solvers(env, orc, solver):
    """The bins' partials of p.q (CG), r_hat.v (BiCGSTAB, CGS) and (t.s, t.t)
    (BiCGSTAB): residual parity on a diagonally dominant system."""
    mxs, ctx, torch = env
    A = I.random_spd(1 << 16, seed=31)
    assert A.nnz >= 1 << 19
    rows = np.repeat(np.arange(A.n), A.row_lengths())
    A.val[rows == A.col] *= 4.0
    b = I.uniform_vector(A.n, 32)
    M = mxs.Matrix.from_host(ctx, A)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    mxs.solve(ctx, solver, M, torch.from_numpy(b).cuda(), x, tol=1e-10)
    xh = x.cpu().numpy()
    slack = 64 * 2.0 ** -53 * np.linalg.norm(np.abs(b) + orc.absrow(A, xh)) / np.linalg.norm(b)
    assert orc.true_relres(A, b, xh) <= 1e-10 + slack


def test_values_refreshed_in_place(env, orc):
    """PageRank's transition values are written after the layout is built."""
    mxs, ctx, torch = env
    G = I.powerlaw_graph(60000, seed=41)
    assert G.nnz >= 1 << 19
    st, xo, _, _ = orc.pagerank(G, 0.85, 1e-12)
    g = mxs.Graph(ctx, G)
    x = torch.zeros(G.n, dtype=torch.float64, device="cuda")
    r = mxs.pagerank(ctx, g, x, 0.85, 1e-12)
    assert st == orc.OK and r.status == mxs.OK
    assert np.abs(x.cpu().numpy() - xo).sum() <= 1e-12


@pytest.mark.parametrize("short", [0, 500])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_hyb_whole_rows(env, orc, dt, short):
    """A hybrid whose ELL part (one slot a row) holds just under and just over
    a quarter of the entries: the products of whole rows and of the COO part's,
    with rows without entries."""
    mxs, ctx, torch = env
    lens = [4, 4, 0, 4] * 70000 + [100] + [1] * short
    A = _matrix(40000, lens, 31)
    ell = int((np.asarray(lens) > 0).sum())
    assert (4 * (A.nnz - ell) >= 3 * A.nnz) == (short == 0)
    B = mxs.Matrix.from_host(ctx, A).convert("hyb", dt, ell_width=1)
    assert B.info()["ell_width"] == 1 and B.info()["coo_nnz"] == A.nnz - ell
    tdt = torch.float64 if dt == "f64" else torch.float32
    tol = 1e-13 if dt == "f64" else 1e-5
    x, y0, val = I.uniform_vector(40000, 32), I.uniform_vector(A.n, 33), A.val
    if dt == "f32":
        x, y0, val = (v.astype(np.float32).astype(np.float64) for v in (x, y0, val))
    R = I.CSRMatrix(A.n, 40000, A.rowptr, A.col, val)
    xd = torch.from_numpy(x).to(tdt).cuda()
    for beta in (0.0, -0.5):
        ya = torch.from_numpy(y0).to(tdt).cuda()
        if beta == 0.0:
            ya.fill_(float("nan"))
        yb = ya.clone()
        mxs.spmv(ctx, B, xd, ya, 1.5, beta)
        mxs.spmv(ctx, B, xd, yb, 1.5, beta, noalloc=True)
        err = np.abs(ya.cpu().numpy().astype(np.float64) - orc.spmv_csr(R, x, 1.5, beta, y0))
        assert (err <= tol * (1.5 * orc.absrow(R, x) + abs(beta * y0)) + 1e-30).all()
        assert torch.equal(ya, yb)
