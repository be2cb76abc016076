"""Runs of a sequence on both sides of the capture: the first with some tensors
are launched, the fifth is captured, the later ones replay the graph.  All give
the first run's maps bit for bit, with eager work, waits and other outputs
between them, on the default stream and another, before and after a selection."""
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,m,kind,replan", [
    (side, 20, kind, replan) for side in (False, True)
    for kind, replan in (("none", False), ("none", True), ("global", True))] + [(False, 512, "none", True)])
def test_runs_agree(side, m, kind, replan):
    from paper_2406_17656_amd import Context, DeviceCSC
    A0h, Ash = P.config4(m=m, nmat=6)
    kw = dict(kind="global", thresh=0.1) if kind == "global" else {}
    ctx = Context(0)
    A0, As = DeviceCSC.from_host(A0h), [DeviceCSC.from_host(A) for A in Ash]
    vals = [A.val for A in As]
    seq = ctx.sequence(A0, As[0], len(As), prec="f32", power=2, replan_each_run=replan, **kw)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if side else torch.cuda.current_stream()
    with torch.cuda.stream(stream):
        sets = [(seq.alloc_maps(), torch.empty(len(As), dtype=torch.float64, device="cuda")) for _ in range(2)]
        junk = torch.randn(1 << 18, device="cuda")
        for order in (None, seq.order()):      # the classes again: the same maps
            if order is not None:
                seq.select(order)
            first = None
            for i, which in enumerate([0] * 7 + [1, 0, 1, 1, 0, 1, 1, 1, 0, 1]):
                Ms, res2 = sets[which]
                for M in Ms:
                    M.zero_()
                res2.fill_(float("nan"))
                junk = junk * 1.0001 + 1.0
                if i % 3 == 0:
                    torch.cuda.synchronize()
                seq.run(vals, Ms, res2)
                got = [M.clone() for M in Ms] + [res2.clone()]
                if first is None:
                    first = got
                    ctx.sync_status()
                assert all(torch.equal(a, b) for a, b in zip(first, got)), (order, i)
    ctx.sync_status()
    seq.close()
    ctx.close()


@pytest.mark.parametrize("replan", [False, True])
def test_callers_capture(replan):
    """A run inside the caller's own capture: its replays give the eager run's maps."""
    from paper_2406_17656_amd import Context, DeviceCSC
    A0h, Ash = P.config4(m=20, nmat=5)
    ctx = Context(0)
    A0, As = DeviceCSC.from_host(A0h), [DeviceCSC.from_host(A) for A in Ash]
    vals = [A.val for A in As]
    seq = ctx.sequence(A0, As[0], len(As), prec="f64", power=2, replan_each_run=replan)
    Ms, res2 = seq.alloc_maps(), torch.empty(len(As), dtype=torch.float64, device="cuda")
    seq.run(vals, Ms, res2)
    want = [M.clone() for M in Ms] + [res2.clone()]
    ctx.sync_status()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        seq.run(vals, Ms, res2)
    junk = torch.randn(1 << 16, device="cuda")
    for i in range(5):
        for M in Ms:
            M.zero_()
        junk = junk * 1.0001 + 1.0
        g.replay()
        if i % 2:
            torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want, Ms + [res2])), i
    for i in range(6):       # and the sequence's own graph, beside it
        res2.zero_()
        seq.run(vals, Ms, res2)
        assert all(torch.equal(a, b) for a, b in zip(want, Ms + [res2])), i
    ctx.sync_status()
    torch.cuda.synchronize()
    del g
    seq.close()
    ctx.close()
