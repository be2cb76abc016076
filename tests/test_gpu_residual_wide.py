"""The explicit residual on columns of many entries: a dense column of A_k, A_0
or M among short ones (taken by the whole wave inside the short ones' kernel),
and matrices whose columns are all long (a wave per column from the start), with
runs around 64 entries, row sets beyond the 768 or 1024 accumulators, and
several windows of 32768 rows."""
import numpy as np
import pytest
import torch

import oracle as O
import pde_inputs as P

pytestmark = pytest.mark.gpu


def columns(n, lens, rng):
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ri = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in lens]).astype(np.int32)
    return P.CSC(n, cp, ri, rng.standard_normal(ri.size))


def residual(Ak, A0, M, prec="f64"):
    """(library, oracle, the second of two calls' device time in ms)"""
    from paper_2406_17656_amd import Context, DeviceCSC
    mv = M.val.astype(np.float32) if prec == "f32" else M.val
    ctx = Context(0)
    args = (DeviceCSC.from_host(Ak), DeviceCSC.from_host(A0), torch.as_tensor(M.colptr).cuda(),
            torch.as_tensor(M.rowind).cuda(), torch.as_tensor(mv).cuda(), prec)
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    first = ctx.residual(*args)[0]
    e[0].record()
    r2 = ctx.residual(*args)[0]
    e[1].record()
    ctx.sync_status()
    assert torch.equal(first, r2)
    want, _ = O.residual(Ak, A0, O.Pattern(Ak.n, M.colptr, M.rowind), mv.astype(np.float64))
    ms = e[0].elapsed_time(e[1])
    ctx.close()
    return float(r2[0]), want, ms


# sums of squares in some order: at most n terms of one sign, n * 1.1e-16 relative on either side, and the
# products in them as much as a column has entries
def bound(n):
    return 4 * n * 1.2e-16


@pytest.mark.parametrize("a_len", [5, 7, 9])   # the forms of 8 lanes, without and with the table, and of 16
@pytest.mark.parametrize("dense", ["A_k", "A_0", "M", "all"])
def test_dense_column(a_len, dense):
    n = 5003 if dense in ("M", "all") else 131101
    rng = np.random.default_rng(a_len)
    mats = {}
    for name, length in (("A_k", a_len), ("A_0", a_len), ("M", 9)):
        lens = np.full(n, length)
        if dense in (name, "all"):
            lens[[7, n // 2, n - 1]] = (n, n - 1, n)
        mats[name] = columns(n, lens, rng)
    got, want, ms = residual(mats["A_k"], mats["A_0"], mats["M"], "f32" if a_len == 7 else "f64")
    assert abs(got - want) <= bound(n) * want
    # a range of a dense column reads what lies in it: some 10 ms; every range reading all of it, seconds
    assert ms < 250.0


@pytest.mark.parametrize("n,a_len,m_len", [
    (63, 63, 63),          # fewer columns and rows than a wave has lanes
    (700, 64, 17),         # runs of 64 entries
    (700, 65, 17),         # and of one more
    (1200, 130, 70),       # more than 64 runs, row sets beyond 1024
    (40009, 33, 40),       # two windows
    (100003, 12, 90),      # four windows, few rows in each
])
def test_long_columns(n, a_len, m_len):
    rng = np.random.default_rng(n + a_len)
    A = columns(n, np.full(n, a_len), rng)
    A0 = columns(n, rng.integers(0, min(2 * a_len, n) + 1, n), rng)
    M = columns(n, rng.integers(0, min(2 * m_len, n) + 1, n), rng)
    assert A.rowind.size * float(M.rowind.size) > 512.0 * n * n
    got, want, _ = residual(A, A0, M)
    assert abs(got - want) <= bound(max(n, 1 << 12)) * want


@pytest.mark.parametrize("entries", [511, 512, 513])
def test_longest_column_of_the_short_form(entries):
    """One column with as many entries as the groups of lanes still take, and
    one more, beside short and empty ones."""
    n = 3001
    rng = np.random.default_rng(entries)
    lens = np.full(n, 4)
    lens[0::9] = 0
    lens[1501] = entries - 5 * 4
    A0 = columns(n, lens, rng)
    A = columns(n, np.full(n, 4), rng)
    M = columns(n, np.full(n, 5), rng)
    got, want, _ = residual(A, A0, M)
    assert abs(got - want) <= bound(n) * want
