"""The adjoint with its scale dL read on the device gives what the host scalar
gives, bit for bit, and scales of other devices and types still work."""
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("scale", [1.0, -0.375])
def test_device_scale(prec, scale):
    from paper_2406_17656_amd import Context, DeviceCSC
    from paper_2406_17656_amd.autograd import SamResidualLoss
    A0h, Ash = P.config2(m=20, nmat=2)
    ctx = Context(0)
    A0, Ak = DeviceCSC.from_host(A0h), DeviceCSC.from_host(Ash[0])
    cp, ri = ctx.pattern(Ak, 2)
    w = torch.linspace(0.2, 1.0, ri.numel(), dtype=torch.float64, device="cuda")
    plan = ctx.plan(Ak, A0, cp, ri)
    want = plan.backward(Ak.val, A0.val, w, 3.0, dL=scale, prec=prec)
    for dL in (torch.tensor(scale, dtype=torch.float64, device="cuda"),
               torch.tensor([scale], dtype=torch.float64, device="cuda"),
               torch.tensor(scale), torch.tensor(scale, device="cuda")):
        got = plan.backward(Ak.val, A0.val, w, 3.0, dL=dL, prec=prec)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    leaf = Ak.val.clone().requires_grad_()
    (scale * SamResidualLoss.apply(plan, leaf, A0.val, w, 3.0, prec)).backward()
    assert torch.equal(leaf.grad, want[0])
    plan.close()
    ctx.close()
