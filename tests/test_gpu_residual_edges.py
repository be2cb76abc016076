"""The explicit residual kernel at the edges of its layout: columns of A_k
longer than its eight lanes, more than eight columns of M per column, row sets
beyond one window (4096 rows) and beyond one pass of accumulators (64 rows),
columns of M or A_0 that are empty, and a number of columns that is no
multiple of eight."""
import numpy as np
import pytest
import torch

import oracle as O
import pde_inputs as P

pytestmark = pytest.mark.gpu


def random_csc(n, lens, rng, span=None):
    """Column j with lens[j] distinct rows, all over the matrix or within
    `span` of the diagonal."""
    rows, cp = [], np.zeros(n + 1, dtype=np.int32)
    for j in range(n):
        lo, hi = (0, n) if span is None else (max(0, j - span), min(n, j + span + 1))
        r = np.sort(rng.choice(hi - lo, size=min(lens[j], hi - lo), replace=False) + lo)
        rows.append(r)
        cp[j + 1] = cp[j] + r.size
    ri = np.concatenate(rows).astype(np.int32)
    return P.CSC(n, cp, ri, rng.standard_normal(ri.size))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,a_len,m_len,span", [
    (1, 1, 1, None),          # one column
    (7, 3, 3, None),          # fewer columns than one wave takes
    (61, 8, 8, None),         # exactly eight entries and eight columns
    (203, 9, 9, 40),          # one more of each
    (517, 21, 37, None),      # several batches of both, row sets beyond 64 rows
    (9001, 6, 11, None),      # three windows of 4096 rows
    (5003, 17, 5, 4500),      # two windows, long columns
])
def test_residual_edges(n, a_len, m_len, span, prec):
    from paper_2406_17656_amd import Context, DeviceCSC
    rng = np.random.default_rng(n)
    Ak = random_csc(n, rng.integers(1, a_len + 1, n), rng, span)
    A0 = random_csc(n, rng.integers(0, a_len + 1, n), rng, span)
    M = random_csc(n, rng.integers(0 if n > 7 else 1, m_len + 1, n), rng, span)
    mv = M.val.astype(np.float32) if prec == "f32" else M.val
    ctx = Context(0)
    r2, a02 = ctx.residual(DeviceCSC.from_host(Ak), DeviceCSC.from_host(A0), torch.as_tensor(M.colptr).cuda(),
                           torch.as_tensor(M.rowind).cuda(), torch.as_tensor(mv).cuda(), prec)
    ctx.sync_status()
    r2o, a2o = O.residual(Ak, A0, O.Pattern(n, M.colptr, M.rowind), mv.astype(np.float64))
    # sums of squares of generic values, at most 40 + 2500 terms deep: 3e-13 relative
    assert abs(float(r2.cpu()[0]) - r2o) <= 1e-12 * r2o
    assert abs(float(a02.cpu()[0]) - a2o) <= 1e-12 * max(a2o, 1e-300)
    ctx.close()
