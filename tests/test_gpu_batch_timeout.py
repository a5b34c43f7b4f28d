"""Barrier waits that end before the other workgroups arrive (one poll, so that
every wait of more than a fraction of a microsecond does): a persistent launch
reports the lost state, and the autotuner restores the state, keeps to ordinary
launches and leaves the batch usable."""
import numpy as np
import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    from paper_1608_04118_amd import binding
    return binding


# the persistent launch of single steps, and of pairs of steps
CASES = {"f64": [I.cavity_small(nx=n, ny=70, precision=I.FP64) for n in (64, 96, 130)],
         "f16s": [I.cavity_small(nx=n, ny=70, precision=I.FP16S) for n in (64, 96, 130)],
         "f32_pairs": [I.cavity_small(nx=512, ny=512, precision=I.FP32, Ra=ra) for ra in (1e4, 2e4)]}


def _same(B, batch, ps, steps):
    for i, p in enumerate(ps):
        lat = B.Lattice(p).step(steps)
        a, b = batch.macros(i), lat.macros()
        for k in a:
            assert np.array_equal(a[k], b[k]), (i, k)
        lat.close()


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("mode", [0, 1])
def test_autotune_does_without_persistent_launches(B, case, mode):
    ps = CASES[case]
    b = B.Batch(ps).step(10)
    b.set_mode(mode)
    chunks = b.chunks().tolist()
    b.set_spin_limit(1)
    assert b.autotune(reps=2) > 0
    assert b.info()["persistent"] == 0 and b.chunks().tolist() == chunks
    b.step(7)
    _same(B, b, ps, 17)
    b.close()


@pytest.mark.parametrize("case", CASES)
def test_lost_state_is_reported(B, case):
    ps = CASES[case]
    b = B.Batch(ps)
    b.set_mode(1)
    b.set_spin_limit(1)
    b.step(40)
    for call in (lambda: b.macros(0), lambda: b.nusselt(0), lambda: b.autotune(reps=2)):
        with pytest.raises(B.LtneError) as e:
            call()
        assert e.value.code == B.LBM_EHIP
    b.close()


def test_default_limit_is_restored_by_zero(B):
    ps = CASES["f64"]
    b = B.Batch(ps)
    b.set_mode(1)
    b.set_spin_limit(1)
    b.set_spin_limit(0)
    b.step(20)
    _same(B, b, ps, 20)
    b.close()
