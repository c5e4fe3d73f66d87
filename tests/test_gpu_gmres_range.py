"""GMRES over the range of FP64: a system and a right-hand side scaled by powers
of two.  No step of the method rounds differently then (products, sums, square
roots and quotients of scaled numbers are the scaled results while squares stay
normal numbers, which 2^-400 and 2^400 leave room for), so the steps are the
same and x is the unscaled solve's x times a power of two, bit for bit."""
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


def _solve(env, A, b, scale_a, scale_b):
    mxs, ctx, torch = env
    S = I.CSRMatrix(A.n, A.ncols, A.rowptr, A.col, np.ldexp(A.val, scale_a))
    M = mxs.Matrix.from_host(ctx, S)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    r = mxs.solve(ctx, "gmres", M, torch.from_numpy(np.ldexp(b, scale_b)).cuda(), x, tol=1e-9,
                  restart=12, raise_on_error=False)
    M.close()
    return r, x.cpu().numpy()


@pytest.mark.parametrize("scale_a,scale_b", [(-400, 300), (400, -300), (-400, -300), (400, 300),
                                             (-400, 0), (400, 0), (0, -400), (0, 400)])
def test_scaled_system(env, scale_a, scale_b):
    mxs = env[0]
    A = I.convdiff3d(14)
    b = I.uniform_vector(A.n, 51)
    r0, x0 = _solve(env, A, b, 0, 0)
    assert r0.status == mxs.OK and r0.restarts > 0
    r, x = _solve(env, A, b, scale_a, scale_b)
    assert (r.status, r.iters, r.restarts) == (mxs.OK, r0.iters, r0.restarts)
    assert np.array_equal(x, np.ldexp(x0, scale_b - scale_a))
