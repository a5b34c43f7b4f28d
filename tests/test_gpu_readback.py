"""Reading the macros back: at the edges of the pinned chunks (fields smaller
than one, ending inside one, one value past several, more chunks than the ring
holds), into arrays off a page and with fields left out; bit for bit against a
copy of the device's own memory."""
import ctypes as C

import numpy as np
import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu

FIELDS = ("rho", "ux", "uy", "Tf", "Ts")
# 262144 doubles are one chunk, 524288 pay for a second thread
SIZES = [(5, 4), (229, 229), (512, 512), (4, 65537), (1024, 513), (1100, 1501), (2048, 1700)]


@pytest.fixture(scope="module")
def B():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1608_04118_amd import binding
    return binding


def _params(nx, ny, form):
    return I.cavity_small(nx=nx, ny=ny, precision=form, body_force=(1e-5, -2e-5))


def _read(fn, h, n, wanted, shift):
    """The fields through the C entry, at `shift` doubles into their memory;
    the doubles around them keep their value."""
    mem = [np.full(n + shift + 3, -7.0) for _ in FIELDS]
    ptr = [m[shift:].ctypes.data_as(C.POINTER(C.c_double)) if f in wanted else None for f, m in zip(FIELDS, mem)]
    assert fn(h, *[C.cast(p, C.c_void_p) for p in ptr]) == 0
    for f, m in zip(FIELDS, mem):
        rest = np.concatenate([m[:shift], m[shift + n:]]) if f in wanted else m
        assert (rest == -7.0).all(), f
    return {f: m[shift:shift + n] for f, m in zip(FIELDS, mem) if f in wanted}


@pytest.mark.parametrize("form", [I.FP64, I.FP32], ids=["f64", "f32"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "%dx%d" % s)
def test_fields_arrive(B, form, size):
    import torch
    nx, ny = size
    n, dtype = nx * ny, torch.float64 if form == I.FP64 else torch.float32
    tf = 0.5 + 0.2 * np.random.default_rng(n).uniform(-1, 1, (ny, nx))
    lat = B.Lattice(_params(nx, ny, form), Tf0=tf)
    first = -(-19 * (-(-nx // 64) * 64) * ny * dtype.itemsize // 256) * 256 * 2  # after two population buffers
    mac = lat._pool[first:first + 5 * n * dtype.itemsize].view(dtype).cpu().numpy().astype(np.float64).reshape(5, n)
    assert np.unique(mac[3]).size > n // 4
    fn = B.lib().lbm_ltne_macros
    for wanted, shift in ((FIELDS, 0), (FIELDS, 5), (("ux", "Tf"), 1), (("Ts",), 0), ((), 0)):
        for f, got in _read(fn, lat.h, n, wanted, shift).items():
            assert np.array_equal(got, mac[FIELDS.index(f)]), (f, wanted, shift)
    got = lat.macros()
    for i, f in enumerate(FIELDS):
        assert got[f].shape == (ny, nx) and np.array_equal(got[f].ravel(), mac[i]), f
    lat.close()


def test_batch_reads_lattices_of_any_size_in_any_order(B):
    sizes = [(5, 4), (1100, 700), (64, 64), (229, 229)]
    ps = [_params(nx, ny, I.FP32) for nx, ny in sizes]
    batch = B.Batch(ps).step(3)
    for i in (0, 1, 2, 1, 3, 0):
        lat = B.Lattice(ps[i]).step(3)
        a, b = batch.macros(i), lat.macros()
        for f in FIELDS:
            assert np.array_equal(a[f], b[f]), (i, f)
        lat.close()
    batch.close()
