"""solve_with_map on what the library's steps do not take: a target of another
order or device, a basis that the device has no room for; and numbers of steps
and tolerances that are no plain Python numbers."""
import math

import numpy as np
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2406_17656_amd import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def system(m, seed=0):
    from paper_2406_17656_amd import DeviceCSC
    A0h, Ash = P.config2(m=m, nmat=2)
    b = torch.as_tensor(np.random.default_rng(seed).standard_normal(A0h.n)).cuda()
    return DeviceCSC.from_host(A0h), DeviceCSC.from_host(Ash[0]), b


def generic(ctx, Ak, dinv, b, *args):
    from paper_2406_17656_amd.krylov import SparseOp, gmres
    return gmres(SparseOp(ctx, Ak.n, Ak.colptr, Ak.rowind, Ak.val), lambda v: dinv * v, b, *args)


def test_target_of_another_order(ctx):
    """Refused, but for the order 1, whose diagonal is a number."""
    from paper_2406_17656_amd import DeviceCSC
    from paper_2406_17656_amd.krylov import solve_with_map
    _, Ak, b = system(12)
    for m in (11, 13):
        with pytest.raises(RuntimeError):
            solve_with_map(ctx, Ak, system(m)[0], None, None, None, b)
    one = DeviceCSC(1, torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                    torch.zeros(1, dtype=torch.int32, device="cuda"),
                    torch.full((1,), 4.0, dtype=torch.float64, device="cuda"))
    x, its, hist = solve_with_map(ctx, Ak, one, None, None, None, b, "f64", 1e-8, 20, 200)
    xr, itsr, histr = generic(ctx, Ak, torch.full((1,), 0.25, dtype=torch.float64, device="cuda"), b, 1e-8, 20, 200)
    assert its == itsr and hist == histr and torch.equal(x, xr)


def test_target_on_the_host(ctx):
    from paper_2406_17656_amd import DeviceCSC
    from paper_2406_17656_amd.krylov import solve_with_map
    A0, Ak, b = system(12)
    host = DeviceCSC(A0.n, A0.colptr.cpu(), A0.rowind.cpu(), A0.val.cpu())
    with pytest.raises(RuntimeError):
        solve_with_map(ctx, Ak, host, None, None, None, b)


@pytest.mark.parametrize("restart,maxiter,tol", [
    (np.int64(9), np.int64(30), np.float32(1e-7)),
    (9, 30.0, torch.tensor(1e-7, dtype=torch.float64)),   # cut in the fourth cycle
    (9, 1e4, 1e-7),
    (9, 25.5, 1e-7),                                       # 26 steps
    (40, 25.5, 1e-7),
    (9, math.inf, 1e-7),
])
def test_numbers(ctx, restart, maxiter, tol):
    from paper_2406_17656_amd.krylov import jacobi_diag, solve_with_map
    A0, Ak, b = system(16)
    x, its, hist = solve_with_map(ctx, Ak, A0, None, None, None, b, "f64", tol, restart, maxiter)
    xr, itsr, histr = generic(ctx, Ak, 1.0 / jacobi_diag(A0), b, float(tol), int(restart), maxiter)
    # the same steps but for rounding at the tolerance
    assert abs(its - itsr) <= (1 if itsr < maxiter else 0)
    k = min(len(hist), len(histr)) - 2
    np.testing.assert_allclose(hist[:k], histr[:k], rtol=1e-6)


def test_basis_beyond_the_device(ctx):
    """Room for the few steps that are taken, not for a whole cycle's basis."""
    from paper_2406_17656_amd.krylov import BASIS_BYTES, solve_with_map
    A0, Ak, b = system(400)
    restart = 512
    basis = (2 * restart + 1) * Ak.n * 8
    assert 1 << 30 < basis <= BASIS_BYTES
    want, its, _ = solve_with_map(ctx, Ak, A0, None, None, None, b, "f64", 0.3, restart)
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved(0) + (768 << 20)) / total)
    try:
        x, again, _ = solve_with_map(ctx, Ak, A0, None, None, None, b, "f64", 0.3, restart)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert abs(again - its) <= 1 < its < 200
    # two solutions to the same tolerance, by other roundings: 8 / pi^2 n of them a step
    if again == its:
        assert float(torch.linalg.vector_norm(x - want)) <= 1e-7 * float(torch.linalg.vector_norm(want))
