"""The FP32 classes of four lanes that have a form of eight lanes for few
columns, on both sides of the number of columns at which the forms change, on
blocks that fill the class and that miss it by one row and column."""
import numpy as np
import pytest
import torch

import oracle as O
import pde_inputs as P
from parity_util import TOL, colmax_rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2406_17656_amd import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def blocks(n, rows, cols, longest, rng):
    """Block-diagonal A of order n (the last block ragged) with columns of up to
    `longest` entries, and the pattern that gives every column the first `cols`
    columns of its block."""
    local, lens = [], []
    for j in range(rows):
        must = [j] + [j + cols * i for i in range(1, rows) if j < cols and j + cols * i < rows]
        must = must[:longest]
        rest = np.setdiff1d(np.arange(rows), must)
        r = np.sort(np.append(must, rng.choice(rest, min(longest - len(must), rest.size), replace=False)))
        local.append(r)
        lens.append(r.size)
    nb = -(-n // rows)
    ri = (np.concatenate(local)[None] + rows * np.arange(nb)[:, None]).ravel()
    col = np.repeat(np.arange(nb * rows), np.tile(lens, nb))
    keep = (col < n) & (ri < n)
    ri, col = ri[keep], col[keep]
    cp = np.concatenate([[0], np.cumsum(np.bincount(col, minlength=n))]).astype(np.int32)
    A = P.CSC(n, cp, ri.astype(np.int32), rng.standard_normal(ri.size) + 8.0 * (ri == col))
    sr = (np.arange(n) // rows * rows)[:, None] + np.arange(cols)[None]
    ok = sr < n
    return A, O.Pattern(n, np.concatenate([[0], np.cumsum(ok.sum(1))]).astype(np.int32), sr[ok].astype(np.int32))


@pytest.mark.parametrize("cls,columns", [(5, 8192), (6, 8192), (7, 24576), (8, 16384)])
@pytest.mark.parametrize("past", [False, True])
@pytest.mark.parametrize("miss", [0, 1])
def test_forms_of_a_class(ctx, cls, columns, past, miss):
    from paper_2406_17656_amd import DeviceCSC, autotune
    v = autotune.menu("f32")[cls]
    rng = np.random.default_rng(cls)
    n = columns + past
    A, S = blocks(n, v["max_rows"] - miss, v["NC"] - miss, 9, rng)
    A0, _ = blocks(n, v["max_rows"] - miss, v["NC"] - miss, 5, rng)
    dA, dA0 = DeviceCSC.from_host(A), DeviceCSC.from_host(A0)
    plan = ctx.plan(dA, dA0, torch.as_tensor(S.colptr).cuda(), torch.as_tensor(S.rowind).cuda())
    plan.select([cls], "f32")
    M, _, r = plan.build(dA.val, dA0.val, "f32")
    ctx.sync_status()
    Mo, rho, _, _ = O.sam_build(A, A0, S)
    assert colmax_rel(M.cpu().numpy().astype(np.float64), Mo, S.colptr)[0] <= TOL["f32"]
    assert np.isclose(float(r.cpu()[0]), rho.sum(), rtol=1e-9)
    plan.close()
