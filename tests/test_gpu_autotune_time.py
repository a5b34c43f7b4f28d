"""The autotuner's trials take the steps that its description says: a call lasts
about as long as those steps, of which the persistent launch's are the most."""
import time

import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_call_lasts_as_long_as_its_trials():
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    from paper_1608_04118_amd import binding as B

    def seconds(fn):
        torch.cuda.synchronize()
        t = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        return time.perf_counter() - t

    b = B.Batch([I.cavity_small(nx=512, ny=512, precision=I.FP32, Ra=ra) for ra in (1e4, 2e4)])
    reps, n = 200, 300
    per_step = []
    for mode in (0, 1):
        b.set_mode(mode)
        b.step(20)
        per_step.append(min(seconds(lambda: b.step(n)) for _ in range(3)) / n)
    b.set_mode(0)
    b.step(1)
    single = min(seconds(lambda: [b.step(1) for _ in range(n)]) for _ in range(3)) / n
    # tile widths: the start and three widths; chunk heights: the start and four
    # others, and the mode's own; the ordinary launches
    trials = 4 * (reps + 1) * single + 6 * (2 * reps + 2) * per_step[1] + (2 * reps + 10) * per_step[0]
    took = min(seconds(lambda: b.autotune(reps=reps)) for _ in range(2))
    b.close()
    print("autotune %.1f ms, its trials %.1f ms (persistent step %.1f us)" % (1e3 * took, 1e3 * trials, 1e6 * per_step[1]))
    assert per_step[1] > 2 * per_step[0]  # the persistent launch's steps are the larger part
    assert took < 1.6 * trials + 0.02
