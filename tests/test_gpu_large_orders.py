"""Calls on orders at which the lanes of a row or column, counted together,
exceed 31 and 32 bits: nearly empty matrices with entries at the ends and on
both sides of the powers of two."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2406_17656_amd import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def rows_of(n):
    """A few rows: the ends and the neighbours of 2^27, 2^28, 2^29 and 2^30."""
    r = {0, 1, n - 2, n - 1} | {p + d for b in (27, 28, 29, 30) for p in (1 << b,) for d in (-1, 0, 1)}
    return np.array(sorted(x for x in r if 0 <= x < n))


def pointers(n, rows):
    """n + 1 pointers of a matrix with one entry in each of `rows`."""
    p = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    for i, r in enumerate(rows):
        p[int(r) + 1:(int(rows[i + 1]) + 1 if i + 1 < len(rows) else n + 1)] = i + 1
    return p


def nonzeros(x):
    """The positions of x's nonzero entries, piece by piece."""
    step = 1 << 28
    out = [torch.nonzero(x[i:i + step]).flatten() + i for i in range(0, x.numel(), step)]
    return torch.cat(out).cpu().numpy()


@pytest.mark.parametrize("n,steps", [((1 << 29) + 5, 2), ((1 << 30) + 77, 1), ((1 << 31) - 1, 1)])
def test_product_and_gmres_steps(ctx, n, steps):
    """A and N diagonal on a few rows: the product, the Arnoldi steps and their
    solution touch these rows alone."""
    from paper_2406_17656_amd import _capi as C
    from paper_2406_17656_amd.sam import _buf, _ptr, _size
    rows = rows_of(n)
    k = len(rows)
    rng = np.random.default_rng(k)
    a, m, d, v = (rng.uniform(1.0, 2.0, k) for _ in range(4))
    v /= np.linalg.norm(v)
    at, A, N, two = (torch.as_tensor(x).cuda() for x in (rows, a, m, np.array([2.0])))
    rp, ci = pointers(n, rows), at.to(torch.int32)
    V = torch.zeros((steps + 1, n), dtype=torch.float64, device="cuda")
    V[0, at] = torch.as_tensor(v).cuda()
    x = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
    ctx.apply((rp, ci, None), A, V[0], "f64", y=x, permuted=True)
    assert np.array_equal(nonzeros(x), rows)
    assert np.array_equal(x[at].cpu().numpy(), a * v)
    x.fill_(0.0)
    x[at] = torch.as_tensor(d).cuda()
    Z = torch.full((steps, n), float("nan"), dtype=torch.float64, device="cuda")
    H = torch.empty((steps, steps + 1), dtype=torch.float64, device="cuda")
    state = torch.empty(2 * steps + 3, dtype=torch.float64, device="cuda")
    nb = _size(ctx.lib.sam_gmres_workspace_size, n, steps)
    ws = _buf(nb, "cuda")
    for M in (None, m):
        nrp, nci, nv = (None, None, None) if M is None else (rp, ci, N)
        ctx.check(ctx.lib.sam_gmres_steps(
            ctx.h, n, _ptr(rp), _ptr(ci), _ptr(A), _ptr(nrp), _ptr(nci), _ptr(nv), C.SAM_PREC_F64, _ptr(x), steps, 0,
            steps, 1.0, 0.0, _ptr(V), _ptr(Z), _ptr(H), _ptr(state), _ptr(ws), nb, ctx.stream()))
        assert state.tolist()[0] == steps
        basis = [v]
        for i in range(steps):
            z = (d if M is None else M * d) * basis[i]
            w = a * z
            for _ in range(2):
                w = w - sum((b @ w) * b for b in basis)
            w /= np.linalg.norm(w)
            # each step loses at most the digits that the subtraction of parts of unit size cancels
            # (norms above 0.05 here), and the first's error goes through the second
            for got, want in ((Z[i], z), (V[i + 1], w)):
                assert np.array_equal(nonzeros(got), rows)
                np.testing.assert_allclose(got[at].cpu().numpy(), want, rtol=0, atol=1e-12)
            basis.append(w)
    z0 = Z[0, at].cpu().numpy()
    ctx.check(ctx.lib.sam_gmres_solution(ctx.h, n, 1, _ptr(two), _ptr(Z), _ptr(x), ctx.stream()))
    assert np.array_equal(nonzeros(x), rows)
    np.testing.assert_allclose(x[at].cpu().numpy(), d + 2.0 * z0, rtol=1e-15)
    ctx.sync_status()
    del V, Z, x, ws, rp
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [(1 << 28) + 33, (1 << 29) + 33, (1 << 31) - 1])
def test_row_view_and_topk(ctx, n):
    """One entry in each of a few columns, rows in descending order: the row
    view turns them round, and the selection keeps the candidates that k lets
    in."""
    cols = rows_of(n)
    k = len(cols)
    cp = pointers(n, cols)
    ri = torch.as_tensor(cols[::-1].copy()).cuda().to(torch.int32)
    rp, ci, pm = ctx.apply_prepare(n, cp, ri)
    assert torch.equal(rp, cp)
    assert np.array_equal(ci.cpu().numpy(), cols[::-1])
    assert np.array_equal(pm.cpu().numpy(), np.arange(k)[::-1])
    del rp, ci, pm
    w = torch.ones(k, dtype=torch.float64, device="cuda")
    w[1::2] = 0.5
    for top, kept in ((1, np.arange(k)), (0, np.arange(0, k, 2))):
        got_cp, got_ri = ctx.pattern_topk(cp, ri, w, torch.arange(float(k), dtype=torch.float64, device="cuda"), top)
        assert torch.equal(got_cp, pointers(n, cols[kept]))
        assert np.array_equal(got_ri.cpu().numpy(), cols[::-1][kept])
    ctx.sync_status()
    del cp, got_cp
    torch.cuda.empty_cache()
