"""The classes of a plan and of a sequence read back: selecting them again, also
completed with the rest of the menu, gives the same buckets and the same maps;
an order that was selected is the one read."""
import pytest
import torch

import pde_inputs as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_plan_order(prec):
    from paper_2406_17656_amd import Context, DeviceCSC, autotune
    A0h, Ash = P.config4(m=24, nmat=2)
    ctx = Context(0)
    A0, Ak = DeviceCSC.from_host(A0h), DeviceCSC.from_host(Ash[0])
    cp, ri = ctx.pattern(Ak, 2)
    plan = ctx.plan(Ak, A0, cp, ri)
    own, columns = plan.order(prec), plan.info()["bucket_cols"]
    assert 1 <= len(own) <= 16 and len(set(own)) == len(own)
    M, _, r = plan.build(Ak.val, A0.val, prec)
    n = len(autotune.menu(prec))
    for order in (list(range(n)), own, autotune.complete(own, prec)):
        plan.select(order, prec)
        assert plan.order(prec) == order
        again, _, r2 = plan.build(Ak.val, A0.val, prec)
        if order[:len(own)] == own:
            assert torch.equal(again, M) and torch.equal(r, r2)
            if prec == "f32":
                assert plan.info()["bucket_cols"][:len(columns)] == columns
    plan.close()
    ctx.close()


@pytest.mark.parametrize("kind", ["none", "column"])
def test_sequence_order(kind):
    from paper_2406_17656_amd import Context, DeviceCSC, autotune
    A0h, Ash = P.config3(m=8)
    ctx = Context(0)
    A0, As = DeviceCSC.from_host(A0h), [DeviceCSC.from_host(A) for A in Ash]
    kw = dict(kind=kind, tau=0.85) if kind == "column" else {}
    seq = ctx.sequence(A0, As[0], len(As), prec="f32", power=2, replan_each_run=True, **kw)
    own = seq.order()
    assert own and len(set(own)) == len(own)
    res = []
    for order in (None, list(range(len(autotune.menu("f32")))), own, autotune.complete(own, "f32")):
        if order is not None:
            seq.select(order)
            assert seq.order() == order
        Ms, res2 = seq.alloc_maps(), torch.zeros(len(As), dtype=torch.float64, device="cuda")
        for M in Ms:
            M.zero_()
        seq.run([A.val for A in As], Ms, res2)
        ctx.sync_status()
        res.append((Ms, res2))
    for Ms, res2 in res[2:]:
        assert torch.equal(res2, res[0][1]) and all(torch.equal(a, b) for a, b in zip(Ms, res[0][0]))
    seq.close()
    ctx.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("grid,small", [((8, 8, 8), False), ((40, 40, 40), True)])
def test_rule_sequence_has_classes_for_thin_columns(grid, small, prec):
    """What a rule leaves is not known when a sequence is made: at 64000 columns
    some class is made for columns that keep little, beside one for the whole
    63 x 25 block; few columns have one class for all."""
    from paper_2406_17656_amd import Context, DeviceCSC, autotune
    A0h, Ash = P.config3(m=grid[0])
    ctx = Context(0)
    A0, Ak = DeviceCSC.from_host(A0h), DeviceCSC.from_host(Ash[0])
    seq = ctx.sequence(A0, Ak, 1, prec=prec, power=2, kind="column", tau=0.6, replan_each_run=True)
    menu = autotune.menu(prec)
    cells = [menu[i]["max_rows"] * menu[i]["NC"] for i in seq.order()]
    assert max(cells) >= 63 * 25
    # the narrowest class is at most a quarter of the block, where there is one
    assert min(cells) <= 63 * 25 // 4 if small else len(cells) == 1
    if small and prec == "f64":
        assert min(cells) <= 16 * 8    # 0.16 ns a column against 6.8
    seq.close()
    ctx.close()
