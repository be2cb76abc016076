"""The explicit residual's row table: rows far apart, tables that are nearly
empty, nearly full and overfull (the bitmap takes over inside the same wave),
in the eight- and the sixteen-lane form, every column's own sum."""
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


@pytest.mark.parametrize("n,a_len,m_max,wide", [
    (9001, 7, 1, False),      # a few rows a column
    (9001, 7, 9, False),      # up to 71 rows for 64 slots
    (40009, 7, 16, False),    # up to 120; ten windows
    (8209, 16, 8, True),      # up to 144 rows for 128 slots
    (30011, 16, 32, True),    # up to 528
    (211, 16, 32, True),      # 211 rows at most, one window
])
def test_row_table(n, a_len, m_max, wide):
    from paper_2406_17656_amd import Context, DeviceCSC
    rng = np.random.default_rng(n + m_max)
    Ak = columns(n, np.full(n, a_len), rng)
    A0 = columns(n, rng.integers(0, 9, n), rng)
    M = columns(n, rng.integers(0, m_max + 1, n), rng)
    assert wide == (a_len > 7 or M.rowind.size > 14 * n)
    ctx = Context(0)
    got = [ctx.residual(DeviceCSC.from_host(Ak), DeviceCSC.from_host(A0), torch.as_tensor(M.colptr).cuda(),
                        torch.as_tensor(M.rowind).cuda(), torch.as_tensor(M.val).cuda(), "f64") for _ in range(2)]
    ctx.sync_status()
    want, _ = O.residual(Ak, A0, O.Pattern(n, M.colptr, M.rowind), M.val)
    # squares of sums of at most 33 products, then sums of 528 squares and of n columns (pairwise on both
    # sides): below 600 roundings of 1.1e-16 relative to a sum of positive terms
    assert abs(float(got[0][0].cpu()[0]) - want) <= 1e-12 * want
    assert float(got[0][0].cpu()[0]) == float(got[1][0].cpu()[0])
    ctx.close()
