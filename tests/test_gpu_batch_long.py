"""A batch call of more than 2^20 steps, which the library splits: the steps
keep their numbers (they seed the stochastic rounding), so the result is that
of the same steps in two calls, and that of the lattice alone."""
import numpy as np
import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_calls_past_a_million_steps_equal_shorter_ones():
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    from paper_1608_04118_amd import binding as B
    n, more = 1 << 20, 60
    # periodic, so that no walls drain it over so many steps
    p = I.cavity_small(nx=8, ny=8, precision=I.FP16S, periodic_x=1, periodic_y=1, L=8.0, dT=1.0, Ra=100.0, nu_f=0.1,
                       T_init_f=0.3, T_init_s=0.35)
    one = B.Batch([p]).step(n + more)
    two = B.Batch([p]).step(n).step(more)
    alone = B.Lattice(p).step(n + more)
    a, b, c = one.macros(0), two.macros(0), alone.macros()
    for k in a:
        assert np.array_equal(a[k], b[k]) and np.array_equal(a[k], c[k]), k
    assert np.isfinite(a["Tf"]).all()
    one.close()
    two.close()
    alone.close()
