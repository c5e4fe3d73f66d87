"""Where the iterative solvers stop, with the host some iterations ahead of the
device: an iteration limit on either side of the counts that the kernels send
is met exactly, and x does not depend on how far ahead the host may run."""
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


@pytest.mark.parametrize("kind", ["cg", "pcg", "pipecg", "bicgstab", "cgs", "gmres"])
@pytest.mark.parametrize("limit", [1, 3, 4, 5, 8, 9, None])
def test_stops(env, orc, kind, limit):
    mxs, ctx, torch = env
    A = I.poisson3d(21)             # more rows than one work-group takes
    b = I.uniform_vector(A.n, 5)
    M = mxs.Matrix.from_host(ctx, A)
    kw = {"restart": 7} if kind == "gmres" else {}
    P = mxs.Precond(ctx, M, "jacobi") if kind == "pcg" else None
    if P:
        kw["precond"] = P
    out = []
    for every in (1, 3, 16, 100):
        x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        r = mxs.solve(ctx, "cg" if P else kind, M, torch.from_numpy(b).cuda(), x, tol=1e-9,
                      max_iters=limit or 20000, check_every=every, raise_on_error=False, **kw)
        if limit:
            assert (r.status, r.iters) == (mxs.NOT_CONVERGED, limit)
        else:
            assert r.status == mxs.OK and r.relres_true <= 1e-9
        out.append((r.iters, x.cpu().numpy()))
    for it, x in out[1:]:
        assert it == out[0][0] and np.array_equal(x, out[0][1])
