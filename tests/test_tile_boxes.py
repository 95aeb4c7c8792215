"""The box shapes of the tile sweep, asked of the library's host code (no GPU):
boxes fit the workgroup and its images, cover the grid, and are dealt to the
XCDs in blocks that are nearly full."""
import ctypes

import pytest

import paper_2004_02833_amd as pm


class Grid(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int) for f in ("nx", "ny", "nz")] + [(f, ctypes.c_longlong) for f in ("ncell", "pstride")]


class Boxes(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int) for f in ("w", "ty", "tz", "nseg", "nty", "ntz", "rowch", "nmain", "whole", "bx", "by", "bz")]


def _boxes(prec, nx, ny, nz):
    n = nx * ny * nz
    t = Boxes()
    f = getattr(pm.lib(), "_ZN2pm9tile_geomEiRKNS_8GridDescERNS_8TileGeomE")
    f.restype = ctypes.c_bool
    assert f(ctypes.c_int(prec), ctypes.byref(Grid(nx, ny, nz, n, (n + 63) // 64 * 64)), ctypes.byref(t))
    return t


@pytest.mark.parametrize("prec", [pm.PM_FP64, pm.PM_FP32])
@pytest.mark.parametrize("ny,nz", [(40, 40), (1, 700), (33, 1)])
def test_boxes_cover_the_grid_in_full_blocks(prec, ny, nz):
    for nx in list(range(1, 200)) + list(range(200, 9000, 37)):
        t = _boxes(prec, nx, ny, nz)
        assert t.w * t.ty * t.tz <= 512
        assert (t.ty * t.tz + t.ty + t.tz) * t.rowch <= (476 if prec == pm.PM_FP64 else 264)
        assert (t.nseg - 1) * t.w < nx <= t.nseg * t.w and (t.nty - 1) * t.ty < ny <= t.nty * t.ty and (t.ntz - 1) * t.tz < nz <= t.ntz * t.tz
        # places of a row of blocks against its segments: 9 in two blocks of 5 is the worst
        assert -(-t.nseg // t.bx) * t.bx * 9 <= 10 * t.nseg, (nx, t.nseg, t.bx)
