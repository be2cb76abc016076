"""The library's GMRES steps beyond 262144 rows, where a block's chunk holds more
rows than the block takes at once, with maps of both precisions, against the
driver on callables (modified Gram-Schmidt)."""
import numpy as np
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [512, 513, 560])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_against_the_callables(m, prec):
    from paper_2406_17656_amd import Context, DeviceCSC
    from paper_2406_17656_amd.krylov import SparseOp, gmres, jacobi_diag, solve_with_map
    A0h, Ash = P.config2(m=m, nmat=2)
    ctx = Context(0)
    A0, Ak = DeviceCSC.from_host(A0h), DeviceCSC.from_host(Ash[0])
    b = torch.as_tensor(np.random.default_rng(m).standard_normal(A0h.n)).cuda()
    cp, ri = ctx.pattern(Ak, 1)
    M, _, _ = ctx.build(Ak, A0, cp, ri, prec)
    ctx.sync_status()
    # two cycles of 12 steps, far from convergence: the projected problems are
    # well conditioned (below 1e3), and a dot product's sums are some 30 additions
    # deep, so x and the residuals agree to 30 * 2^-53 * 24 * 1e3 < 1e-10
    x, its, hist = solve_with_map(ctx, Ak, A0, cp, ri, M, b, prec=prec, tol=1e-14, restart=12, maxiter=24)
    A = SparseOp(ctx, Ak.n, Ak.colptr, Ak.rowind, Ak.val)
    N = SparseOp(ctx, Ak.n, cp, ri, M, prec)
    d = jacobi_diag(A0)
    xr, itr, hr = gmres(A, lambda v: N(v / d), b, 1e-14, 12, 24)
    assert its == itr == 24 and len(hist) == len(hr)
    assert float(torch.linalg.vector_norm(x - xr) / torch.linalg.vector_norm(xr)) <= 1e-10
    assert np.allclose(hist, hr, rtol=1e-10, atol=0.0)
    ctx.close()
