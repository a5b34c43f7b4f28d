"""Fields read into one and the same array: it holds the last of them, as when
the fields are copied one after another; the other arrays are not affected."""
import ctypes as C

import numpy as np
import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu

# two chunks a field and two threads; many chunks and eight threads
SIZES = [(1024, 257), (1100, 1501)]


@pytest.mark.parametrize("form", [I.FP64, I.FP32], ids=["f64", "f32"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "%dx%d" % s)
def test_array_shared_by_fields_holds_the_last(form, size):
    from paper_1608_04118_amd import binding as B
    nx, ny = size
    n = nx * ny
    rng = np.random.default_rng(n)
    lat = B.Lattice(I.cavity_small(nx=nx, ny=ny, precision=form, body_force=(1e-5, -2e-5)),
                    Tf0=0.5 + 0.2 * rng.uniform(-1, 1, (ny, nx)), Ts0=0.5 + 0.2 * rng.uniform(-1, 1, (ny, nx)))
    lat.step(2)
    want = {k: v.ravel() for k, v in lat.macros().items()}
    ptr = lambda a: C.c_void_p(a.ctypes.data)
    fn = B.lib().lbm_ltne_macros
    for _ in range(4):
        a, b, c = (np.empty(n) for _ in range(3))
        assert fn(lat.h, ptr(a), ptr(b), ptr(a), ptr(c), ptr(c)) == 0
        assert np.array_equal(a, want["uy"]) and np.array_equal(b, want["ux"]) and np.array_equal(c, want["Ts"])
    # two arrays that overlap in half: the later field is whole, the other's other half is
    h = n // 2
    a = np.empty(n + h)
    assert fn(lat.h, None, ptr(a), None, ptr(a[h:]), None) == 0
    assert np.array_equal(a[h:], want["Tf"]) and np.array_equal(a[:h], want["ux"][:h])
    lat.close()
