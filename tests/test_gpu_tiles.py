"""Two and three steps per launch over tiles: every precision form, at the edges of the
tiles (a last tile of one or two nodes, a single tile, the smallest lattices,
periodic wraps inside one tile), bit for bit against single steps; and a batch
of such lattices against the lattices alone."""
import numpy as np
import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu

FORMS = {"f64": I.FP64, "f32": I.FP32, "f16s": I.FP16S, "f32sr": I.FP32SR}
# nx, ny, periodic_x, periodic_y
SIZES = [(4, 4, 0, 0), (3, 3, 1, 1), (5, 4, 0, 0), (4, 3, 0, 1), (9, 5, 1, 0), (33, 17, 0, 0), (65, 49, 0, 1),
         (129, 130, 1, 1), (257, 6, 0, 0), (6, 257, 1, 0), (385, 193, 0, 0)]


@pytest.fixture(scope="module")
def B():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1608_04118_amd import binding
    return binding


def _case(nx, ny, px, py, form, seed=0):
    rng = np.random.default_rng(seed + nx * 1000 + ny)
    p = I.cavity_small(nx=nx, ny=ny, precision=form, periodic_x=px, periodic_y=py, Hv=40.0, body_force=(1e-5, -2e-5),
                       wall_thermal=(0, 1, 1, 0), T_wall=(1.0, 0.0, 0.0, 0.2), L=32.0, dT=1.0, Ra=1e4)
    phi = 0.55 + 0.1 * rng.uniform(-1, 1, (ny, nx))
    hv = 40.0 * (1 + 0.4 * rng.uniform(-1, 1, (ny, nx)))
    tf, ts = (0.5 + 0.2 * rng.uniform(-1, 1, (ny, nx)) for _ in range(2))
    return p, phi, hv, tf, ts


def _same(a, b):
    for k in a:
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "%dx%d_p%d%d" % s)
def test_tiles_equal_single_steps(B, form, size):
    p, phi, hv, tf, ts = _case(*size, FORMS[form])
    for fields in (dict(phi=phi, Hv=hv, Tf0=tf, Ts0=ts), dict(Tf0=tf, Ts0=ts), dict(phi=phi), dict(Hv=hv)):
        one, many = B.Lattice(p, **fields), B.Lattice(p, **fields)
        for calls in ((4, 3), (8,), (2,)):  # 2 + 2, 3; 3 + 3 + 2; 2
            for n in calls:
                many.step(n)
            for _ in range(sum(calls)):
                one.step(1)
            _same(one.macros(), many.macros())
        one.close()
        many.close()


# one workgroup, tiles of a node's halo across both ends of an axis, the
# longest halo a periodic axis takes, the largest lattices of the rule, the
# first beyond it
SMALL = [(8, 8, 1, 1), (7, 40, 1, 0), (40, 5, 0, 1), (64, 64, 0, 0), (100, 37, 1, 1), (192, 191, 0, 0),
         (257, 193, 0, 0), (384, 384, 1, 0), (386, 385, 0, 0)]


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("size", SMALL, ids=lambda s: "%dx%d_p%d%d" % s)
def test_small_lattices_equal_single_steps(B, form, size):
    p, phi, hv, tf, ts = _case(*size, FORMS[form])
    for fields in (dict(phi=phi, Hv=hv, Tf0=tf, Ts0=ts), dict(Tf0=tf, Ts0=ts), dict(phi=phi), dict(Hv=hv)):
        one, many = B.Lattice(p, **fields), B.Lattice(p, **fields)
        for calls in ((8, 7), (9,), (25,), (4,)):  # 8, 7; 5 + 4; 7 + 6 + 6 + 6; 4 (of eight)
            for n in calls:
                many.step(n)
            for _ in range(sum(calls)):
                one.step(1)
            _same(one.macros(), many.macros())
        one.close()
        many.close()


@pytest.mark.parametrize("form", FORMS)
def test_batch_tiles_equal_single_lattices(B, form):
    cases = [_case(*s, FORMS[form]) for s in SIZES]
    batch = B.Batch([c[0] for c in cases], phi_fields=[c[1] if i % 2 else None for i, c in enumerate(cases)])
    batch.step(6)
    batch.step(5)
    for i, c in enumerate(cases):
        lat = B.Lattice(c[0], phi=c[1] if i % 2 else np.full(c[1].shape, c[0]["phi"]))
        for _ in range(11):
            lat.step(1)
        _same(lat.macros(), batch.macros(i))
        lat.close()
    batch.close()


@pytest.mark.parametrize("form", ["f64", "f32", "f32sr"])
@pytest.mark.parametrize("size", [s for s in SIZES if not (s[2] and s[3])], ids=lambda s: "%dx%d_p%d%d" % s)
def test_adjoint_tiles_equal_single_sweeps(B, form, size):
    """Segments of one step take single recorded steps and single sweeps;
    longer ones the launches of several steps and of two sweeps."""
    p, phi, hv, tf, ts = _case(*size, FORMS[form])
    for n, every in ((2, 0), (7, 0), (12, 4)):
        out = []
        for k in (1, every):
            lat = B.Lattice(p, phi=phi, Hv=hv, Tf0=tf, Ts0=ts)
            lat.step(1)
            out.append(lat.adjoint(n, ckpt_every=k) + (lat.macros(),))
            lat.close()
        a, b = out
        assert a[0] == b[0] and np.abs(a[1]).max() > 0
        assert np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
        _same(a[3], b[3])
