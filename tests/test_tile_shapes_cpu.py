"""Tile shapes of the launches of two and three steps, on the host: they cover
the lattice, fit the kernel's LDS slots, and waste little of their last tiles
also on lattices that are thin or just past a multiple of the usual shape."""
import ctypes as C
import random

import pytest

from paper_1608_04118_amd import binding as B
from paper_1608_04118_amd import inputs as I

SLOTS = {I.FP64: 536, I.FP32: 1072, I.FP16S: 2144, I.FP32SR: 1072}  # as the kernels'
CUS = 256


class Grid(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("w", "h", "ntx", "ntiles", "per_xcd")]


def tile_grid(nx, ny, precision, nsub, px=0, py=0):
    fn = getattr(B.lib(), "_ZN4ltne9tile_gridERK15lbm_ltne_paramsi")
    fn.restype, fn.argtypes = Grid, [C.c_void_p, C.c_int]
    p = B.params_from_dict(I.cavity_small(nx=nx, ny=ny, precision=precision, periodic_x=px, periodic_y=py))
    return fn(C.byref(p), nsub)


def ceil(a, b):
    return -(-a // b)


def busiest(w, h, nx, ny, nsub):
    """Wavefront passes of the CU with the most tiles."""
    per_tile = sum(ceil((w + 2 * g) * (h + 2 * g), 64) for g in range(nsub))
    return ceil(ceil(nx, w) * ceil(ny, h), CUS) * per_tile


def least(nx, ny, precision, nsub):
    """The fewest passes over tiles of every width, each as tall as fits or split evenly."""
    g2, out = 2 * (nsub - 1), None
    for w in range(4, 257):
        hmax = SLOTS[precision] // (w + g2) - g2
        if hmax < 4:
            break
        for h in {hmax, max(4, min(hmax, ceil(ny, ceil(ny, hmax))))}:
            c = busiest(w, h, nx, ny, nsub)
            out = c if out is None else min(out, c)
    return out


def sizes():
    r = random.Random(3)
    out = [(400000, 6), (100000, 5), (49, 40000), (55, 40000), (25, 80000), (40000, 50), (97, 20000), (4096, 4096)]
    for _ in range(12):
        nx = int(4 * (30000 / 4) ** r.random())
        out.append((nx, max(4, int(1e6 * 20 ** r.random() / nx))))
    return out


@pytest.mark.parametrize("precision", sorted(SLOTS))
@pytest.mark.parametrize("nsub", [2, 3])
def test_shapes(precision, nsub):
    for nx, ny in sizes():
        g = tile_grid(nx, ny, precision, nsub)
        assert g.ntx == ceil(nx, g.w) and g.ntiles == g.ntx * ceil(ny, g.h) and g.per_xcd == ceil(g.ntiles, 8)
        assert (g.w + 2 * (nsub - 1)) * (g.h + 2 * (nsub - 1)) <= SLOTS[precision]
        # 4/3 by the rule, and the even splits that it compares with are within 1.1 of the fewest
        assert busiest(g.w, g.h, nx, ny, nsub) <= 1.47 * least(nx, ny, precision, nsub), (nx, ny, g.w, g.h)
