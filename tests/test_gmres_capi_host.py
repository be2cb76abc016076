"""Argument checks of the GMRES calls: before any device work, in order."""
import ctypes

import pytest

from paper_2406_17656_amd import _capi as C

WS = ctypes.c_void_p(1 << 20)


@pytest.fixture()
def hctx():
    lib = C.load()
    h = ctypes.c_void_p()
    assert lib.sam_create(ctypes.byref(h), C.SAM_NO_DEVICE) == C.SAM_OK
    yield lib, h
    lib.sam_destroy(h)


def steps(lib, h, n=4, Arp=1, Aci=1, Av=1, Nrp=1, Nci=1, Nv=1, prec=0, d=1, restart=3, first=0, count=3, V=1, Z=1,
          H=1, state=1, ws=WS, nb=None):
    if nb is None:
        size = ctypes.c_size_t()
        lib.sam_gmres_workspace_size(max(n, 1), min(max(restart, 1), 512), ctypes.byref(size))
        nb = size.value
    return lib.sam_gmres_steps(h, n, Arp, Aci, Av, Nrp, Nci, Nv, prec, d, restart, first, count, 1.0, 1e-8, V, Z, H,
                               state, ws, nb, None)


def test_workspace_size(hctx):
    lib, _ = hctx
    nb = ctypes.c_size_t()
    for n, restart in ((0, 5), (-1, 5), (4, 0), (4, C.SAM_GMRES_MAX_RESTART + 1)):
        assert lib.sam_gmres_workspace_size(n, restart, ctypes.byref(nb)) == C.SAM_ERR_ARG
    assert lib.sam_gmres_workspace_size(4, 5, None) == C.SAM_ERR_ARG
    assert lib.sam_gmres_workspace_size((1 << 31) - 1, 512, ctypes.byref(nb)) == C.SAM_OK and nb.value > 8 * (1 << 31) - 16


@pytest.mark.parametrize("bad", [
    dict(n=0), dict(restart=0), dict(restart=513), dict(first=-1), dict(count=-1), dict(first=4), dict(first=2, count=2),
    dict(prec=7), dict(Arp=None), dict(Aci=None), dict(Av=None), dict(Nci=None), dict(Nv=None), dict(d=None),
    dict(V=None), dict(Z=None), dict(H=None), dict(state=None), dict(ws=None), dict(nb=8),
])
def test_steps(hctx, bad):
    lib, h = hctx
    assert steps(lib, h, **bad) == C.SAM_ERR_ARG


def test_steps_reach_the_device(hctx):
    lib, h = hctx
    assert steps(lib, h) == C.SAM_ERR_UNSUPPORTED
    assert steps(lib, h, Nrp=None, Nci=None, Nv=None) == C.SAM_ERR_UNSUPPORTED
    assert steps(lib, None) == C.SAM_ERR_ARG


def test_solution(hctx):
    lib, h = hctx
    assert lib.sam_gmres_solution(h, 0, 1, 1, 1, 1, None) == C.SAM_ERR_ARG
    assert lib.sam_gmres_solution(h, 4, -1, 1, 1, 1, None) == C.SAM_ERR_ARG
    for k in range(3):
        assert lib.sam_gmres_solution(h, 4, 2, *[None if i == k else 1 for i in range(3)], None) == C.SAM_ERR_ARG
    assert lib.sam_gmres_solution(h, 4, 2, 1, 1, 1, None) == C.SAM_ERR_UNSUPPORTED
