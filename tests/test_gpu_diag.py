"""Products over diagonals (matrices of few of them, any format) against the
CPU oracle where the form can go wrong: the smallest matrices that take it,
last slices that are not full, numbers of diagonals with and without a last
round, threes of neighbouring diagonals, shifts that leave x on either side,
holes, too many sets of diagonals; its dot products inside the solvers and its
values refreshed in place.

Chains of additions: 64 diagonals on 4 accumulators and 2 more, 18 roundings:
2e-15 of sum |a||x| in FP64, 1.1e-6 in FP32, within the library's 1e-13 and
1e-5."""
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


def _diagonals(n, ncols, offs, seed, keep=None):
    """Every entry (i, i + o) inside the matrix; keep(i, k): a mask of the rows
    that have diagonal k."""
    i = np.arange(n)[:, None]
    c = i + np.sort(np.asarray(offs, np.int64))[None, :]
    on = (c >= 0) & (c < ncols)
    if keep is not None:
        on &= keep(i, np.arange(len(offs))[None, :])
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(on.sum(1), out=rp[1:])
    return I.CSRMatrix(n, ncols, rp.astype(np.int32), c[on].astype(np.int32),
                       I.rng(seed).uniform(-1, 1, int(rp[-1])))


def _revalued(A, seed):
    A.val[:] = I.rng(seed).uniform(-1, 1, A.nnz)
    return A


MATRICES = {
    # (matrix, whether it takes the form)
    "5pt_163": lambda: (_revalued(I.poisson2d(163), 1), True),     # 132193 entries
    "5pt_162": lambda: (_revalued(I.poisson2d(162), 1), False),    # 130572: below 2^17
    "27pt_18": lambda: (_revalued(I.stencil27(18), 2), True),
    "7pt_29": lambda: (_revalued(I.poisson3d(29), 3), True),
    # threes without a whole last round; no threes; a round of 8 and a rest
    "threes_12": lambda: (_diagonals(20001, 20001, [-900, -899, -898, -1, 0, 1, 70, 71, 72,
                                                    500, 501, 502], 4), True),
    "diag_13": lambda: (_diagonals(10177, 10177, list(range(-30, 35, 5)), 5), True),
    "diag_64": lambda: (_diagonals(2117, 2117, range(-32, 32), 6), True),
    "diag_65": lambda: (_diagonals(2117, 2117, range(-32, 33), 6), False),
    # wider and taller than square, offsets that leave x on either side
    "wide": lambda: (_diagonals(20000, 21000, [-3, 0, 1, 2, 900, 999, 1000], 7), True),
    "tall": lambda: (_diagonals(25003, 25000, [-40, -3, -2, -1, 0, 1], 8), True),
    # holes: every ninth row lacks a diagonal (within a fifth), every second
    # all but one (beyond)
    "holes": lambda: (_diagonals(30000, 30000, [-7, -1, 0, 1, 7], 9,
                                 lambda i, k: (i % 9 != 0) | (k != 1)), True),
    "many_holes": lambda: (_diagonals(60000, 60000, [-7, -1, 0, 1, 7], 9,
                                      lambda i, k: (i % 2 == 0) | (k == 2)), False),
    # a tenth of the entries of ten diagonals missing at random: too many sets
    "sets": lambda: (_diagonals(20000, 20000, range(-9, 10), 10,
                                lambda i, k: (k > 9) | (I.rng(43).random((len(i), 19)) > 0.1)),
                     False),
    "empty_rows": lambda: (_diagonals(50003, 50003, [-1, 0, 1], 11,
                                      lambda i, k: i % 20 != 0), True),
}


@pytest.mark.parametrize("name", sorted(MATRICES))
def test_products(env, orc, name):
    mxs, ctx, torch = env
    A, takes = MATRICES[name]()
    M = mxs.Matrix.from_host(ctx, A)
    x, y0 = I.uniform_vector(A.ncols, 12), I.uniform_vector(A.n, 13)
    for fmt, dt in (("csr", "f64"), ("csr", "f32"), ("csr", "f16"), ("coo", "f64"),
                    ("coo", "f32"), ("ell", "f64"), ("ell", "f32"), ("hyb", "f64")):
        B = M.convert(fmt, dt)
        vb = {"f64": 8, "f32": 4, "f16": 2}[dt]
        if fmt in ("csr", "coo"):   # the second copy of the values
            own = A.nnz * (vb + 8) if fmt == "coo" else A.nnz * (vb + 4) + 4.1 * A.n
            assert (B.info()["bytes"] > own + 0.9 * A.nnz * vb) == takes, (fmt, dt)
        tdt = torch.float64 if dt == "f64" else torch.float32
        val, xr, yr = A.val, x, y0
        if dt != "f64":
            xr, yr = (v.astype(np.float32).astype(np.float64) for v in (x, y0))
            val = orc.cast_f32(A.val)[1].astype(np.float64)
        if dt == "f16":
            _, h, s = orc.rowscale_f16(A)
            val = orc.f16_bits_to_f64(h) * np.repeat(s.astype(np.float64), A.row_lengths())
        R = I.CSRMatrix(A.n, A.ncols, A.rowptr, A.col, val)
        tol = 1e-13 if dt == "f64" else 1e-5
        xd = torch.from_numpy(xr).to(tdt).cuda()
        y = torch.from_numpy(yr).to(tdt).cuda()
        mxs.spmv(ctx, B, xd, y, 1.5, -0.5)
        scale = orc.absrow(R, xr)
        err = np.abs(y.cpu().numpy().astype(np.float64) - orc.spmv_csr(R, xr, 1.5, -0.5, yr))
        assert (err <= tol * (1.5 * scale + 0.5 * np.abs(yr)) + 1e-30).all(), (fmt, dt)
        # beta = 0 never reads y; the allocation-free product is the same bits
        ya, yb = (torch.full((A.n,), float("nan"), dtype=tdt, device="cuda") for _ in range(2))
        mxs.spmv(ctx, B, xd, ya)
        mxs.spmv(ctx, B, xd, yb, noalloc=True)
        err = np.abs(ya.cpu().numpy().astype(np.float64) - orc.spmv_csr(R, xr))
        assert (err <= tol * scale + 1e-30).all() and torch.equal(ya, yb), (fmt, dt)
        B.close()


def test_nonfinite_x_stays_in_its_rows(env):
    """Holes and shifts outside x never bring in a value of another column."""
    mxs, ctx, torch = env
    for name in ("5pt_163", "27pt_18", "wide", "tall", "holes"):
        A, _ = MATRICES[name]()
        M = mxs.Matrix.from_host(ctx, A)
        x = torch.ones(A.ncols, dtype=torch.float64, device="cuda")
        cols = [0, 1, 63, 64, A.ncols // 2, A.ncols - 2, A.ncols - 1]
        x[cols[::2]] = float("nan")
        x[cols[1::2]] = float("inf")
        y = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        mxs.spmv(ctx, M, x, y)
        rows = np.repeat(np.arange(A.n), A.row_lengths())
        assert np.array_equal(np.flatnonzero(~np.isfinite(y.cpu().numpy())),
                              np.unique(rows[np.isin(A.col, cols)])), name


@pytest.mark.parametrize("solver", ["cg", "bicgstab", "cgs", "gmres", "pipecg"])
def test_inside_solvers(env, orc, solver):
    """The product's dot-product partials (p.q; r_hat.v; t.s and t.t): residual
    parity on grids whose last work-group and slice are not full."""
    mxs, ctx, torch = env
    A = I.poisson3d(31) if solver in ("cg", "pipecg") else I.convdiff3d(31)
    rows = np.repeat(np.arange(A.n), A.row_lengths())
    A.val[rows == A.col] += 0.5
    b = I.uniform_vector(A.n, 32)
    M = mxs.Matrix.from_host(ctx, A)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    mxs.solve(ctx, solver, M, torch.from_numpy(b).cuda(), x, tol=1e-10)
    xh = x.cpu().numpy()
    slack = 64 * 2.0 ** -53 * np.linalg.norm(np.abs(b) + orc.absrow(A, xh)) / np.linalg.norm(b)
    assert orc.true_relres(A, b, xh) <= 1e-10 + slack


def test_many_slices_a_work_group(env, orc):
    """More work-groups than dot partials (2^20 + 200 rows): several slices each."""
    mxs, ctx, torch = env
    A = _diagonals((1 << 20) + 200, (1 << 20) + 200, [-1, 0, 1], 41)
    rows = np.repeat(np.arange(A.n), A.row_lengths())
    A.val[:] = np.where(rows == A.col, 3.0, -1.0)
    b = I.uniform_vector(A.n, 42)
    M = mxs.Matrix.from_host(ctx, A)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    mxs.solve(ctx, "cg", M, torch.from_numpy(b).cuda(), x, tol=1e-10)
    assert orc.true_relres(A, b, x.cpu().numpy()) <= 1.001e-10


def test_values_refreshed_in_place(env, orc):
    """PageRank's transition values are written after the form is built: a grid
    whose cells link to their four neighbours."""
    mxs, ctx, torch = env
    P = I.poisson2d(200)
    rows = np.repeat(np.arange(P.n), P.row_lengths())
    off = rows != P.col
    G = I.inlinks(P.n, P.col[off], rows[off])
    assert G.nnz >= 1 << 17
    st, xo, _, _ = orc.pagerank(G, 0.85, 1e-12)
    g = mxs.Graph(ctx, G)
    x = torch.zeros(G.n, dtype=torch.float64, device="cuda")
    r = mxs.pagerank(ctx, g, x, 0.85, 1e-12)
    assert st == orc.OK and r.status == mxs.OK
    assert np.abs(x.cpu().numpy() - xo).sum() <= 1e-12
