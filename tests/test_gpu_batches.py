"""Batches of steps whose substeps queued too few sweeps: a substep call over a tiny time
step before the batch makes the context expect fewer sweeps of that substep (Subsystem I,
II or the adjoint I) than its steps need, so the first step of the batch ends on the host
and the steps behind it are queued again.

The reference takes the same state in a new context, with its default expectations.
Tolerance: both stop the same fixed points at 1e-13; steps differ by that and by the
rounding of sums over another particle order, states are of order 1: 1e-11.
"""
import numpy as np
import pytest

import paper_2203_06513_amd as ec
import workloads

pytestmark = pytest.mark.gpu

BAR = 1e-11


def close(g, s, L):
    assert set(g) == set(s)
    for k in g:
        d = np.asarray(g[k]) - np.asarray(s[k])
        if k == "x":
            d = np.mod(d + L / 2, L) - L / 2
        assert np.abs(d).max() <= BAR * max(1.0, np.abs(s[k]).max()), k


@pytest.mark.parametrize("steps", [2, 9, 19])   # within a batch, and past one (8 symmetric steps, 16 others)
@pytest.mark.parametrize("short", ["I", "II", "adjoint", "all"])
@pytest.mark.parametrize("spin", [False, True])
@pytest.mark.parametrize("splitting", [0, 1])
def test_batch_with_too_few_sweeps_queued(splitting, spin, short, steps):
    w = workloads.get("paper52" if spin else "paper51").scaled(n_particles=3000)
    arr = workloads.generate(w)
    tiny = 1e-9 * w.dt
    kw = dict(map=ec.MAP_SEIDEL, splitting=splitting)
    with ec.Context.from_workload(w, **kw) as c:
        c.load(arr)
        if short in ("I", "all"):
            assert c.substep_particles(tiny)[0] <= 2
        if short in ("adjoint", "all"):
            assert c.substep_particles_adjoint(tiny)[0] <= 2
        if short in ("II", "all"):
            assert c.substep_fields(tiny)[0] <= 2
        s0 = c.state()
        rc, done, kI, kII, _ = c.step(steps)
        g = c.state()
    assert rc == 0 and done == steps
    with ec.Context.from_workload(w, **kw) as c:
        c.load(s0, solve_gauss=False)
        rc, done, rI, rII, _ = c.step(steps)
        s = c.state()
    assert rc == 0 and done == steps
    assert kI.tolist() == rI.tolist() and kII.tolist() == rII.tolist()
    assert min(kI) > 2 and min(kII) > 2   # more than the tiny substeps needed
    close(g, s, w.L)


@pytest.mark.parametrize("spin", [False, True])
@pytest.mark.parametrize("splitting", [0, 1])
def test_failing_batch_leaves_its_start(splitting, spin):
    """No step of a batch converges within the allowed sweeps: the state stays, bit by bit."""
    w = workloads.get("paper52" if spin else "paper51").scaled(n_particles=3000)
    with ec.Context.from_workload(w, map=ec.MAP_SEIDEL, splitting=splitting, max_iter=3) as c:
        c.load(workloads.generate(w))
        before = c.state()
        rc, done, *_ = c.step(20, check=False)
        after = c.state()
    assert rc == ec.ENOTCONV and done == 0
    for k in before:
        np.testing.assert_array_equal(before[k], after[k])
