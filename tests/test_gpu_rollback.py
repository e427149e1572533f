"""Steps that fail and are rolled back: what the context keeps for the steps after them."""
import numpy as np
import pytest

import paper_2203_06513_amd as ec
import workloads

pytestmark = pytest.mark.gpu


def beams(spin, M):
    """Two cold beams on one lattice, in any order, in a uniform transverse potential: no
    current and no charge, so an explicit start of Subsystem I is its fixed point to
    rounding (a residual of order 1e-16, where another particle's increment leaves 0.03),
    while Subsystem II needs 5 iterations at this step and tolerance (contraction about
    dt^2 / 8)."""
    n = 100 * M
    w = workloads.get("paper52" if spin else "paper51").scaled(M=M, L=0.25 * M, n_particles=n, dt=0.1, tol=1e-13)
    arr = dict(workloads.generate(w))
    x = (np.arange(n // 2) + 0.5) * w.L / (n // 2)
    p = np.random.default_rng(3).choice([0.3, -0.3], n // 2)
    arr["x"], arr["p"] = np.concatenate([x, x]), np.concatenate([p, -p])
    for k, v in (("ey", 0.0), ("ez", 0.0), ("ay", 1.5), ("az", 0.7)):
        arr[k] = np.full(M, v)
    return w, arr


@pytest.mark.parametrize("M", [32, 160])
@pytest.mark.parametrize("spin", [False, True])
@pytest.mark.parametrize("splitting", [0, 1])
def test_failed_fields_leave_no_previous_start(splitting, spin, M):
    """Subsystem I commits, Subsystem II does not converge: the increments that the commit
    kept are of an order that is undone, so the next substep starts explicitly, at its
    fixed point, and not from other particles' increments."""
    w, arr = beams(spin, M)
    with ec.Context.from_workload(w, map=ec.MAP_SEIDEL, splitting=splitting, warmstart=ec.WS_PREVIOUS,
                                  max_iter=3) as c:
        c.load(arr)
        c.substep_particles()
        before = c.state()
        rc, done, *_ = c.step(2, check=False)
        after = c.state()
        assert rc == ec.ENOTCONV and done == 0
        for k in before:
            np.testing.assert_array_equal(before[k], after[k])
        c.substep_particles()
        assert c.last_res_hist_I[0] < 1e-12


@pytest.mark.parametrize("M", [64, 160])
@pytest.mark.parametrize("splitting", [0, 1])
def test_failed_first_step_leaves_no_previous_start(splitting, M):
    """No sweep of the first step converges: nothing has been committed yet, so the next
    substep starts explicitly, as in a new context."""
    w = workloads.get("paper51").scaled(M=M, n_particles=3000)
    kw = dict(map=ec.MAP_SEIDEL, splitting=splitting, warmstart=ec.WS_PREVIOUS, max_iter=3, sweep_guess=1)
    out = []
    for fail in (True, False):
        with ec.Context.from_workload(w, **kw) as c:
            c.load(workloads.generate(w))
            if fail:
                rc, done, *_ = c.step(1, check=False)
                assert rc == ec.ENOTCONV and done == 0
            k = c.substep_particles(1e-3 * w.dt)[0]
            out.append((k, c.state()))
    assert out[0][0] == out[1][0]
    for k in out[0][1]:
        np.testing.assert_array_equal(out[0][1][k], out[1][1][k])


# (splitting, spin, M, dt, sigma, amplitude, hbar, tol, allowed sweeps, what fails): runs whose
# need grows past the allowed sweeps at some step, in the oracle's counts at steps 4, 12, 0; 3,
# 15, 0 (closing substep alone); 9, 10, 2 (plain steps: Subsystem I; II); 10, 15, 17 (with spin)
GROWING = [
    (1, False, 32, 0.1, 0.08, 0.0, 0.0, 1e-12, 4, "closing"),
    (1, False, 160, 0.05, 0.3, 0.0, 0.0, 1e-13, 4, "closing"),
    (1, False, 160, 0.1, 0.08, 0.0, 0.0, 3e-12, 4, "closing"),
    (1, True, 32, 0.1, 0.15, 0.0, 1e-5, 1e-12, 4, "closing"),
    (1, True, 160, 0.05, 0.3, 0.0, 1e-5, 1e-13, 4, "closing"),
    (1, True, 160, 0.1, 0.08, 0.0, 1e-5, 3e-12, 4, "closing"),
    (0, False, 32, 0.05, 0.08, 0.0, 0.0, 1e-12, 4, "I"),
    (0, False, 160, 0.05, 0.3, 0.0, 0.0, 1e-11, 4, "I"),
    (0, False, 32, 0.1, 0.3, 0.3, 0.0, 3e-12, 5, "II"),
    (0, True, 32, 0.05, 0.08, 0.0, 1e-5, 1e-12, 4, "I"),
    (0, True, 160, 0.05, 0.3, 0.0, 1e-5, 1e-11, 4, "I"),
    (0, True, 32, 0.1, 0.3, 0.3, 1e-2, 3e-12, 5, "II"),
]


@pytest.mark.parametrize("guess", [0, 1])   # the default, and too few sweeps queued at first
@pytest.mark.parametrize("splitting,spin,M,dt,sigma,amplitude,hbar,tol,allowed,what", GROWING)
def test_failing_step_leaves_the_step_before(splitting, spin, M, dt, sigma, amplitude, hbar, tol, allowed, what,
                                             guess):
    """The steps before a failing one stand and its own start is put back, bit for bit (e_x and
    the item list too, which the closing adjoint substep writes over), and what is run
    from there is what a context that took only those steps runs."""
    steps = 24
    w = workloads.get("paper52" if spin else "paper51").scaled(
        M=M, L=0.25 * M, n_particles=2000, dt=dt, sigma=sigma, amplitude=amplitude, hbar=hbar, tol=tol)
    arr = workloads.generate(w)
    kw = dict(map=ec.MAP_SEIDEL, splitting=splitting, sweep_guess=guess)
    with ec.Context.from_workload(w, **kw) as c:
        c.load(arr)
        _, _, kI, kII, _ = c.step(steps)
        need = dict(I=kI, II=kII, closing=c.last_sweeps_I2)
    over = {k: np.flatnonzero(v > allowed) for k, v in need.items()}
    j = min(v[0] for v in over.values() if len(v))
    assert [k for k, v in over.items() if len(v) and v[0] == j] == [what]
    out = []
    for fail in (True, False):
        with ec.Context.from_workload(w, **dict(kw, **(dict(max_iter=allowed) if fail else {}))) as c:
            c.load(arr)
            rc, done, *_ = c.step(steps if fail else int(j), check=False)
            assert rc == (ec.ENOTCONV if fail else 0) and done == j
            states = [c.state()]
            c.substep_particles(0.1 * dt)
            c.substep_fields(0.1 * dt)
            c.substep_particles_adjoint(0.1 * dt)
            out.append(states + [c.state()])
    for a, b in zip(*out):
        for k in a:
            np.testing.assert_array_equal(a[k], b[k], err_msg=k)
