"""The autotuner's decisions on a plan that only keeps the order it was given
(no GPU): what it reuses and what it compares."""
import pytest
import torch

from paper_2406_17656_amd import autotune


class Plan:
    """Refuses the orders in `refused`; starts with the order `first`."""

    nnz_S = 70

    def __init__(self, first=(3,), refused=()):
        self.selected, self.refused, self.selects = list(first), [list(r) for r in refused], 0
        self.ctx = type("Ctx", (), {"device": 0})()

    def info(self):
        return {"n": 10, "max_rows": 25, "max_cols": 13, "gathered": 350}

    def order(self, prec):
        return list(self.selected)

    def select(self, order, prec):
        self.selects += 1
        if list(order) in self.refused:
            raise autotune.SamError(8, "some column fits no listed variant")
        self.selected = list(order)


@pytest.fixture(autouse=True)
def cpu(monkeypatch, tmp_path):
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda device: "gpu")
    monkeypatch.setattr(autotune, "CACHE", str(tmp_path / "tune.json"))
    # the fewer of the menu's first classes stand in front, the faster
    monkeypatch.setattr(autotune, "_time", lambda plan, *a: 10.0 + (16 - plan.selected[0]))


def test_cached_order_of_another_menu_is_not_reused(monkeypatch):
    plan = Plan()
    first = autotune.tune(plan, None, None, "f32")
    again = autotune.tune(plan, None, None, "f32")
    assert not first["cached"] and again["cached"] and again["order"] == first["order"]
    menu = autotune.menu("f32")
    for key in ("G", "R", "NC", "TC"):
        other = [dict(v) for v in menu]
        other[2][key] += 1
        monkeypatch.setattr(autotune, "menu", lambda prec="f32", weighted=0, m=other: m)
        assert not autotune.tune(plan, None, None, "f32")["cached"]


def test_cached_order_that_is_refused_is_tuned_again():
    best = autotune.tune(Plan(), None, None, "f32")["order"]
    plan = Plan(refused=[best])
    res = autotune.tune(plan, None, None, "f32")
    assert not res["cached"] and res["order"] != best and plan.selected == res["order"]


def test_plan_keeps_its_classes_where_they_are_fastest(monkeypatch):
    """No order of the menu's first-variant family is as fast as the classes that
    the plan came with."""
    own = [5, 3, 9]
    monkeypatch.setattr(autotune, "_time", lambda plan, *a: 5.0 if plan.selected[:3] == own else 9.0)
    plan = Plan(first=own)
    res = autotune.tune(plan, None, None, "f32", use_cache=False)
    assert res["order"][:3] == own and res["us"] == 5.0 and plan.selected == res["order"]


def test_sequence_keeps_its_classes_where_they_are_fastest(monkeypatch):
    own = [5, 3, 9]

    class Seq(Plan):
        n_src, now = 2, 0.0

        def order(self):
            return list(self.selected)

        def select(self, order):
            Plan.select(self, order, "f32")

        def alloc_maps(self):
            return []

        def run(self, *a):
            Seq.now += 1.0 if self.selected[:3] == own else 2.0

    import time
    monkeypatch.setattr(time, "perf_counter", lambda: Seq.now)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    seq = Seq(first=own)
    res = autotune.tune_sequence(seq, [torch.zeros(1)], [0], "f32", reps=2)
    assert res["order"][:3] == own and seq.selected == res["order"]


def test_order_calls_validate_arguments():
    import ctypes
    from paper_2406_17656_amd import _capi as C
    lib = C.load()
    out, cnt = (ctypes.c_int32 * 16)(), ctypes.c_int32()
    assert lib.sam_plan_order(None, 1, 16, ctypes.byref(cnt), out) == C.SAM_ERR_ARG
    assert lib.sam_sequence_order(None, 16, ctypes.byref(cnt), out) == C.SAM_ERR_ARG
