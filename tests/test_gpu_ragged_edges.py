"""Top-k selection, row views and structure checks on columns and rows of
lengths around the sixteen lanes, the staged 64 entries and the eight entries of
a check's step, with ties, infinities and NaN in the gradients; exact against
the oracle and numpy."""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu
LENGTHS = [0, 1, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 130, 0, 2]


@pytest.fixture(scope="module")
def ctx():
    from paper_2406_17656_amd import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def pattern(n, seed):
    rng = np.random.default_rng(seed)
    lens = np.minimum(rng.permutation(np.resize(LENGTHS, n)), n)
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ri = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in lens]).astype(np.int32)
    return rng, cp, ri


@pytest.mark.parametrize("n", [1, 15, 16, 17, 200, 1025])
@pytest.mark.parametrize("k", [0, 2, 16, 200])
def test_topk(ctx, n, k):
    rng, cp, ri = pattern(n, n)
    w = rng.choice([1.0, 0.5], ri.size)
    g = rng.integers(-3, 3, ri.size).astype(np.float64)
    g[rng.random(ri.size) < 0.1] = np.nan
    g[rng.random(ri.size) < 0.1] = np.inf
    g[rng.random(ri.size) < 0.1] = -np.inf
    if ri.size == 0:
        pytest.skip("no entries")
    t = [torch.as_tensor(x).cuda() for x in (cp, ri, w, g)]
    got_cp, got_ri = ctx.pattern_topk(*t, k)
    want = O.select_topk(O.Pattern(n, cp, ri), w, g, k)
    assert np.array_equal(got_cp.cpu().numpy(), want.colptr)
    assert np.array_equal(got_ri.cpu().numpy(), want.rowind)


@pytest.mark.parametrize("n", [1, 17, 200, 1025])
def test_row_view(ctx, n):
    """Rows of every length up to n (the first rows are in most columns)."""
    rng = np.random.default_rng(n)
    p = np.linspace(1.0, 0.0, n) ** 4
    mask = rng.random((n, n)) < p[:, None]
    mask[0] = True
    cols = [np.flatnonzero(mask[:, j]) for j in range(n)]
    cp = np.concatenate([[0], np.cumsum([c.size for c in cols])]).astype(np.int32)
    ri = np.concatenate(cols).astype(np.int32)
    rp, ci, pm = (x.cpu().numpy() for x in ctx.apply_prepare(n, torch.as_tensor(cp).cuda(), torch.as_tensor(ri).cuda()))
    col = np.repeat(np.arange(n), np.diff(cp))
    order = np.lexsort((col, ri))
    assert np.array_equal(rp, np.concatenate([[0], np.cumsum(np.bincount(ri, minlength=n))]))
    assert np.array_equal(ci, col[order])
    assert np.array_equal(pm, order)


@pytest.mark.parametrize("length", [1, 2, 7, 8, 9, 16, 17, 33])
@pytest.mark.parametrize("column", [0, 127, 128, 511, 512, 1100])
def test_bad_entries_are_found(ctx, length, column):
    """One column with its last entry repeated, descending, negative or beyond
    n is named; the structure without it passes."""
    from paper_2406_17656_amd import DeviceCSC, SamError
    n = 1101
    lens = np.ones(n, dtype=np.int64)
    lens[column] = length
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ri = np.concatenate([np.arange(length) * 3 if j == column else [j] for j in range(n)]).astype(np.int32)
    val = torch.ones(ri.size, dtype=torch.float64, device="cuda")
    last = cp[column + 1] - 1
    for bad in [None, -1, n] + ([ri[last - 1], ri[last - 1] - 1] if length > 1 else []):
        r = ri.copy()
        if bad is not None:
            r[last] = bad
        A = DeviceCSC(n, torch.as_tensor(cp).cuda(), torch.as_tensor(r).cuda(), val)
        if bad is None:
            ctx.pattern(A, 1)
        else:
            with pytest.raises(SamError, match=f"column {column} "):
                ctx.pattern(A, 1)
