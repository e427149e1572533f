"""Large readouts with the process held to one, two or three processors: the ring is emptied
by no more threads than that, and values come back as they were set."""
import os
import threading
import time

import numpy as np
import pytest

import paper_2203_06513_amd as ec

pytestmark = pytest.mark.gpu

SLOT = 2 << 17   # doubles of a 2 MiB slot of the ring


def threads_now():
    return len(os.listdir("/proc/self/task"))


@pytest.mark.parametrize("cpus", [1, 2, 3])
@pytest.mark.parametrize("n", [3 * SLOT // 2 + 1, 35 * SLOT + 77])
def test_round_trip_on_few_processors(n, cpus):
    had = os.sched_getaffinity(0)
    if len(had) < cpus:
        pytest.skip("fewer processors than the case wants")
    rng = np.random.default_rng(n)
    x, p = rng.uniform(0, 7.9, n), rng.normal(size=n)
    most = []
    with ec.Context(8.0, 64, 3, n, 0.01, 1e-12) as c:
        c.set_particles(x, p)
        c.get_particles()   # the runtime's own threads are started
        base = threads_now() + 1
        for _ in range(5):   # each with a thread that watches
            seen, stop = [0], threading.Event()

            def watch():
                while not stop.is_set():
                    seen[0] = max(seen[0], threads_now())
                    time.sleep(0)

            w = threading.Thread(target=watch)
            w.start()
            try:
                os.sched_setaffinity(0, sorted(had)[:cpus])
                gx, gp = c.get_particles()
            finally:
                os.sched_setaffinity(0, had)
                stop.set()
                w.join()
            most.append(seen[0])
    assert min(most) <= base + cpus   # (a thread of another kind may come up beside one readout)
    assert np.array_equal(gp, p)
    assert np.abs(gx - x).max() <= 4 * np.finfo(float).eps * 8.0
