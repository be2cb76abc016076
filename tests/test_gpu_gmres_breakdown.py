"""The library's Arnoldi steps where a step leaves nothing (an order of 1, an
operator that the preconditioner inverts) and where values are not finite: the
iterations and histories of the driver on callables."""
import math

import numpy as np
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


def both(A0h, Akh, b, *args):
    from paper_2406_17656_amd import Context, DeviceCSC
    from paper_2406_17656_amd.krylov import SparseOp, gmres, jacobi_diag, solve_with_map
    ctx = Context(0)
    A0, Ak = DeviceCSC.from_host(A0h), DeviceCSC.from_host(Akh)
    bd = torch.as_tensor(b).cuda()
    got = solve_with_map(ctx, Ak, A0, None, None, None, bd, "f64", *args)
    dinv = 1.0 / jacobi_diag(A0)
    want = gmres(SparseOp(ctx, Ak.n, Ak.colptr, Ak.rowind, Ak.val), lambda v: dinv * v, bd, *args)
    ctx.close()
    return got, want


def diagonal(d):
    n = d.size
    return P.CSC(n, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), d)


@pytest.mark.parametrize("n", [1, 5, 300])
def test_nothing_left(n):
    rng = np.random.default_rng(n)
    d = rng.uniform(1.0, 2.0, n)
    b = rng.standard_normal(n)
    (x, its, hist), (xr, itsr, histr) = both(diagonal(d), diagonal(d), b, 1e-10, 5, 20)
    assert its == itsr == 1
    assert len(hist) == len(histr) and hist[0] == histr[0] == 1.0
    # one step inverts the matrix: rounding is what is left
    assert hist[-1] <= 1e-14
    np.testing.assert_allclose(x.cpu().numpy(), b / d, rtol=1e-13)


@pytest.mark.parametrize("bad,steps", [(float("nan"), 6),     # no test of the residual ever holds
                                       (float("inf"), 0)])    # inf <= tol inf: done at once
def test_not_finite(bad, steps):
    A0h, Ash = P.config2(m=6, nmat=2)
    b = np.ones(A0h.n)
    b[7] = bad
    (x, its, hist), (xr, itsr, histr) = both(A0h, Ash[0], b, 1e-10, 4, 6)
    assert its == itsr == steps
    assert len(hist) == len(histr)
    assert [math.isfinite(v) for v in hist] == [math.isfinite(v) for v in histr]
    assert torch.equal(torch.isfinite(x), torch.isfinite(xr))
