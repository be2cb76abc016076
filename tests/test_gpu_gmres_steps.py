"""The library's Arnoldi steps against the generic GMRES driver on the same
device operators: the same iterations, residual history and solution to
rounding, at the edges of the steps (fewer rows than a chunk, chunk counts on
both sides of the inline sum, cycles of one step and longer than a tile of
basis vectors, a cycle cut by maxiter, convergence inside a batch)."""
import numpy as np
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32", None])
@pytest.mark.parametrize("m,restart,maxiter", [
    (3, 4, 4),          # n = 9: less than one wave, a short cycle
    (9, 1, 12),         # cycles of one step
    (16, 7, 30),        # n = 256: one full chunk; cut in the fifth cycle
    (17, 20, 2000),     # n = 289: a second chunk of few rows; runs to the tolerance
    (129, 33, 50),      # n = 16641: one chunk more than is summed inline
    (300, 17, 40),      # n = 90000: partials summed by their own launch
])
def test_steps_match_generic_driver(m, restart, maxiter, prec):
    from paper_2406_17656_amd import Context, DeviceCSC
    from paper_2406_17656_amd.krylov import SparseOp, gmres, jacobi_diag, solve_with_map
    A0h, Ash = P.config2(m=m, nmat=2)
    ctx = Context(0)
    A0, Ak = DeviceCSC.from_host(A0h), DeviceCSC.from_host(Ash[0])
    b = torch.as_tensor(np.random.default_rng(m).standard_normal(A0h.n)).cuda()
    cp, ri = ctx.pattern(Ak, 2)
    M = None if prec is None else ctx.build(Ak, A0, cp, ri, prec)[0]
    x, its, hist = solve_with_map(ctx, Ak, A0, cp, ri, M, b, prec or "f64", 1e-9, restart, maxiter)
    dinv = 1.0 / jacobi_diag(A0)
    N = None if M is None else SparseOp(ctx, Ak.n, cp, ri, M, prec)
    apply_M = (lambda v: dinv * v) if N is None else (lambda v: N(dinv * v))
    A = SparseOp(ctx, Ak.n, Ak.colptr, Ak.rowind, Ak.val)
    xr, itsr, histr = gmres(A, apply_M, b, 1e-9, restart, maxiter)
    # both are backward stable: they differ by rounding (1.1e-16) times the condition number (below 1e5
    # here, 8 / pi^2 n) and, per restart, once more
    assert abs(its - itsr) <= (1 if itsr < maxiter else 0)
    k = min(len(hist), len(histr)) - 2
    np.testing.assert_allclose(hist[:k], histr[:k], rtol=1e-6, atol=1e-12)
    if its == itsr:
        assert float(torch.linalg.vector_norm(x - xr)) <= 1e-7 * float(torch.linalg.vector_norm(xr))
    ctx.close()
