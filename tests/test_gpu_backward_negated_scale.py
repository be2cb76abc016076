"""The adjoint's device scale where the tensor is a lazily negated view: the
memory behind it holds the opposite sign."""
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_negated_scale(prec):
    from paper_2406_17656_amd import Context, DeviceCSC
    A0h, Ash = P.config2(m=12, nmat=2)
    ctx = Context(0)
    A0, Ak = DeviceCSC.from_host(A0h), DeviceCSC.from_host(Ash[0])
    cp, ri = ctx.pattern(Ak, 2)
    w = torch.linspace(0.2, 1.0, ri.numel(), dtype=torch.float64, device="cuda")
    plan = ctx.plan(Ak, A0, cp, ri)
    dL = torch.complex(*torch.tensor([0.0, 0.375], dtype=torch.float64, device="cuda")).conj().imag
    assert dL.is_neg() and float(dL) == -0.375
    want = plan.backward(Ak.val, A0.val, w, 3.0, dL=-0.375, prec=prec)
    got = plan.backward(Ak.val, A0.val, w, 3.0, dL=dL, prec=prec)
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    plan.close()
    ctx.close()
