"""What lbm_init_static admits, on the host: exactly the problems whose tiles,
markers and options ask for at most LBM_STATIC_WORKSPACE_BYTES, and none whose
whole workspace is larger than the array behind it. At the largest admitted
problems of the shapes that ask for the most beside that limit (marker lists of
27 entries, where every axis wraps across a last tile of one or two nodes; slip
walls, whose normals come in both body sets; many tiles)."""
import ctypes

import pytest
import torch

from paper_2206_01683_amd import lbm

ARRAY = lbm.STATIC_WORKSPACE_BYTES + (88 << 20)
SHAPES = {
    "lists-of-27": dict(nx=17, ny=18, nz=26, max_active_tiles=1),
    "lists-of-27-slip": dict(nx=17, ny=18, nz=26, max_active_tiles=1, wall_mode=lbm.WALL_SLIP),
    "lists-of-27-implicit": dict(nx=25, ny=17, nz=33, max_active_tiles=1, ib_scheme=lbm.IB_IMPLICIT),
    "tiles": dict(nx=152, ny=96, nz=96),
    "tiles-and-lists": dict(nx=41, ny=33, nz=42),
    "adjoint": dict(nx=128, ny=64, nz=64, with_adjoint=True, max_active_tiles=200),
}


def _counted(p):
    """The bytes that count against the limit, each array rounded up to 256."""
    up = lambda v: (v + 255) // 256 * 256  # noqa: E731
    tiles = ((p.nx + 7) // 8) * ((p.ny + 7) // 8) * ((p.nz + 7) // 8)
    m = max(p.max_markers, 1)
    cap = min(p.max_active_tiles or tiles, tiles) if p.max_markers else 1
    rows, cg = (m + 31) // 32, (m + 255) // 256
    n = 3 * 256 + 3 * up(4 * tiles) + up(4 * cap) + up(8 * m) + up(16 * ((m + 63) // 64 + 8)) + up(32 * rows)
    n += up(8192 * cap) + up(12288 * cap) + up(80 * m) + up(16 * m)
    if p.with_adjoint:
        n += up(6144 * cap) + up(16384 * cap) + up(24 * m) + up(4 * 24 * 16 * p.max_bones) + up(32 * p.ny * p.nz)
    if p.wall_mode == lbm.WALL_SLIP:
        n += up(12 * m)
    if p.ib_scheme == lbm.IB_IMPLICIT:
        n += up(12288 * cap) + up(48 * m) + up(16 * (rows + cg + 34))
    return n


def _admitted(p):
    ctx = ctypes.c_void_p()
    rc = lbm.lib().lbm_init_static(ctypes.byref(ctx), ctypes.byref(p), ctypes.c_void_p(512), ctypes.c_void_p(1024),
                                   None, None, None)
    assert rc in (lbm.ERR_CAPACITY, lbm.ERR_DEVICE)  # no device here: what is admitted ends there
    return rc == lbm.ERR_DEVICE


@pytest.mark.skipif(torch.cuda.is_available(), reason="host check: the buffers are no memory")
@pytest.mark.parametrize("shape", list(SHAPES))
def test_admits_up_to_the_limit_and_fits(shape):
    make = lambda n: lbm.make_params(tau=0.8, max_markers=n, max_bones=4, **SHAPES[shape])  # noqa: E731
    lo, hi = 1, 1 << 24
    assert _counted(make(lo)) <= lbm.STATIC_WORKSPACE_BYTES < _counted(make(hi))
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if _counted(make(mid)) <= lbm.STATIC_WORKSPACE_BYTES else (lo, mid)
    p = make(lo)
    assert _admitted(p) and not _admitted(make(hi))
    assert lbm.lib().lbm_workspace_bytes(ctypes.byref(p)) <= ARRAY
