"""The pinned memory of readbacks is shared by the handles of the process: it
does not grow with their number, serves several threads at once, and goes with
the last handle."""
import threading

import numpy as np
import pytest

from paper_1608_04118_amd import inputs as I

pytestmark = pytest.mark.gpu

NX, NY, N = 1100, 1501, 6  # fields of 13 MB, rings of 24


@pytest.fixture(scope="module")
def B():
    torch = pytest.importorskip("torch")
    assert torch.cuda.is_available()
    from paper_1608_04118_amd import binding
    return binding


def address_space():
    """MB of the process's address space, which pinned memory adds to."""
    with open("/proc/self/status") as f:
        return next(int(line.split()[1]) for line in f if line.startswith("VmSize")) / 1024


def lattices(B):
    return [B.Lattice(I.cavity_small(nx=NX, ny=NY, Ra=1e4 * (i + 1), T_init_f=0.1 * i)).step(i + 1) for i in range(N)]


def test_memory_does_not_grow_with_handles(B):
    import gc
    gc.collect()
    lats = lattices(B)
    out = [np.zeros(NX * NY) for _ in range(5)]
    read = lambda lat: B.lib().lbm_ltne_macros(lat.h, *[a.ctypes.data for a in out])
    for lat in lats[:1] * 3:  # the threads' stacks and arenas as well
        assert read(lat) == 0
    one = address_space()
    for lat in lats[1:]:
        assert read(lat) == 0
    all_read = address_space()
    for lat in lats:
        lat.close()
    closed = address_space()
    print("MB: one handle read %.0f, all %.0f, closed %.0f" % (one, all_read, closed))
    assert all_read - one < 24  # not one more piece
    assert closed < all_read - 15  # it is given back


def test_threads_read_at_the_same_time(B):
    lats = lattices(B)
    want = [lat.macros() for lat in lats]
    got = [[] for _ in lats]
    bad = []

    def work(i):
        try:
            for _ in range(4):
                got[i].append(lats[i].macros())
        except Exception as e:  # shown by the assertion below
            bad.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(N)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for w, reads in zip(want, got):
        for g in reads:
            for k in w:
                assert np.array_equal(w[k], g[k]), k
    for lat in lats:
        lat.close()
