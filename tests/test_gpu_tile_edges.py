"""Launches of two and three steps over the tiles of single lattices too large
for the small-lattice kernel, bit for bit against single steps: lattices whose
last tiles are one and two nodes wide and high, walled and periodic, in every
precision form; both where one tile shape serves all sizes (2048 tiles and
more) and where the shape follows the size; and thin lattices past that rule."""
import ctypes as C

import numpy as np
import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu

FORMS = {"f64": I.FP64, "f32": I.FP32, "f16s": I.FP16S, "f32sr": I.FP32SR}


class Grid(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("w", "h", "ntx", "ntiles", "per_xcd")]


class Small(C.Structure):
    _fields_ = [("grid", Grid), ("steps", C.c_int)]


@pytest.fixture(scope="module")
def B():
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    from paper_1608_04118_amd import binding
    return binding


def _params(nx, ny, form, px=0, py=0):
    return I.cavity_small(nx=nx, ny=ny, precision=form, periodic_x=px, periodic_y=py, Hv=40.0, body_force=(1e-5, -2e-5),
                          wall_thermal=(0, 1, 1, 0), T_wall=(1.0, 0.0, 0.0, 0.2), L=32.0, dT=1.0, Ra=1e4)


def _shape(B, nx, ny, form, nsub):
    """The tiles of a lattice's launches of nsub steps; None: it takes the small-lattice kernel."""
    p = B.params_from_dict(_params(nx, ny, form))
    small = getattr(B.lib(), "_ZN4ltne11small_tilesERK15lbm_ltne_params")
    small.restype, small.argtypes = Small, [C.c_void_p]
    grid = getattr(B.lib(), "_ZN4ltne9tile_gridERK15lbm_ltne_paramsi")
    grid.restype, grid.argtypes = Grid, [C.c_void_p, C.c_int]
    return None if small(C.byref(p)).steps else grid(C.byref(p), nsub)


# sizes with last tiles of one and two nodes along each axis, in launches of two
# and of three steps, under both rules
SIZES = {"f64": [(204, 452), (1962, 50), (2161, 32), (697, 1037), (2817, 301), (3458, 391)],
         "f32": [(1101, 145), (1102, 145), (61, 2627), (311, 534), (2306, 1010), (1345, 2801)],
         "f16s": [(83, 3614), (101, 2989), (1387, 219), (3026, 106), (866, 3722), (994, 2940), (1297, 2438), (1365, 3001)],
         "f32sr": [(1101, 145), (1102, 145), (61, 2627), (311, 534), (721, 2145), (3698, 434)]}


@pytest.mark.parametrize("form", FORMS)
def test_sizes_have_the_edges(B, form):
    missing = {(rule, nsub, axis, r) for rule in ("by size", "one") for nsub in (2, 3) for axis in "xy" for r in (1, 2)}
    for nx, ny in SIZES[form]:
        for nsub in (2, 3):
            g, big = _shape(B, nx, ny, FORMS[form], nsub), _shape(B, 6000, 6000, FORMS[form], nsub)
            rule = "one" if g.ntiles >= 2048 and (g.w, g.h) == (big.w, big.h) else "by size"
            missing -= {(rule, nsub, "x", nx % g.w), (rule, nsub, "y", ny % g.h)}
    assert not missing


def _compare(B, nx, ny, form, px, py):
    rng = np.random.default_rng(nx * 1000 + ny)
    phi = 0.55 + 0.1 * rng.uniform(-1, 1, (ny, nx))
    hv = 40.0 * (1 + 0.4 * rng.uniform(-1, 1, (ny, nx)))
    tf, ts = (0.5 + 0.2 * rng.uniform(-1, 1, (ny, nx)) for _ in range(2))
    p = _params(nx, ny, form, px, py)
    fields = dict(phi=phi, Hv=hv, Tf0=tf, Ts0=ts) if px == py else dict(Tf0=tf, Ts0=ts)
    one, many = B.Lattice(p, **fields), B.Lattice(p, **fields)
    for steps in (6, 5, 2):  # 3 + 3; 3 + 2; 2
        many.step(steps)
        for _ in range(steps):
            one.step(1)
        a, b = one.macros(), many.macros()
        for k in a:
            assert np.array_equal(a[k], b[k]), (k, nx, ny, px, py)
    one.close()
    many.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("px,py", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_last_tiles(B, form, px, py):
    for nx, ny in SIZES[form]:
        print(nx, ny, flush=True)
        _compare(B, nx, ny, FORMS[form], px, py)


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("size", [(60001, 5), (130000, 6), (49, 16001), (57, 30000), (20001, 33)], ids=lambda s: "%dx%d" % s)
def test_thin(B, form, size):
    for px, py in ((0, 0), (1, 1)):
        _compare(B, *size, FORMS[form], px, py)
