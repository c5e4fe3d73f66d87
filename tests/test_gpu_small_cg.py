"""CG on one small system, whose matrix one work-group keeps in registers:
sizes on both sides of each number of threads and rows a thread, rows of the
longest length that a form holds and of one more, rows of unequal length.

The returned x is judged by the oracle's residual, whose rows are accurately
summed: it may exceed the tolerance by the error of the library's own residual
evaluation, 64 u || |b| + |A||x| || (rows of at most 25 entries)."""
import numpy as np
import pytest

from paper_2103_10116_amd import inputs as I

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _spd(n, L, ragged):
    """Symmetric, diagonally dominant, L entries in every row (ragged: fewer in
    every third pair of coupled rows), columns far apart."""
    g = I.rng(n + L)
    i = np.arange(n)
    rows, cols, vals = [], [], []
    for k in range(1, L // 2 + 1):
        far = 2 * k == L
        o = n // 2 if far else (k if k % 2 else n // 2 - k)
        m = i[: n // 2] if far else i
        m = m[m % 3 != 0] if ragged else m
        v = g.uniform(-1, 1, m.size)
        j = (m + o) % n
        rows += [m, j]
        cols += [j, m]
        vals += [v, v]
    A = np.zeros((n, n))
    for r, c, v in zip(rows, cols, vals):
        A[r, c] = v
    A[i, i] = np.abs(A).sum(1) + 0.1 + g.uniform(0, 1, n)
    return I.dense_to_csr(A)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2103_10116_amd import mxs
    ctx = mxs.Context(0)
    yield mxs, ctx, torch
    ctx.close()


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("n,L", [(1, 1), (2, 2), (256, 24), (256, 25), (258, 12), (258, 13),
                                 (1024, 6), (1024, 7), (1026, 6), (1026, 7), (2048, 6),
                                 (2050, 6), (2050, 7), (3074, 5), (3074, 6), (4096, 5),
                                 (4096, 6), (4098, 5)])
def test_small_cg(env, orc, n, L, ragged):
    mxs, ctx, torch = env
    A = _spd(n, L, ragged)
    if not ragged:
        assert np.diff(A.rowptr).max() == L
    b = I.uniform_vector(n, 3)
    M = mxs.Matrix.from_host(ctx, A)
    tol = 1e-10
    for x0 in (np.zeros(n), I.uniform_vector(n, 4)):
        x = torch.from_numpy(x0.copy()).cuda()
        r = mxs.solve(ctx, "cg", M, torch.from_numpy(b).cuda(), x, tol=tol, raise_on_error=False)
        assert r.status == mxs.OK, r
        xh = x.cpu().numpy()
        slack = 64 * U * np.linalg.norm(np.abs(b) + orc.absrow(A, xh)) / np.linalg.norm(b)
        rel = orc.true_relres(A, b, xh)
        assert rel <= tol + slack, (rel, r)
        assert abs(rel - r.relres_true) <= 1e-3 * tol + slack
