"""GPU parity of the 2D passes where their paths meet: rows of particles that stay in
their cell next to rows that cross, at particle counts around a row of 64 and one block
of the re-sort, on grids narrower than a tile; substeps that end in fewer sweeps than
the ones before; solves at the smallest and the largest grids of each kernel.

Tolerance: both sides stop their fixed points at 1e-13 on the same maps, whose
contraction here is below 1/2, so states agree to a few 1e-13 absolute; the fields are
of order 0.01 to 1, hence 1e-11 relative, the bar of the other 2D parity tests.
"""
import numpy as np
import pytest

import paper_2203_06513_amd as ec
from oracle.twod import Oracle2D, initial_state2d
from workloads.twod import generate2d, get2d

pytestmark = pytest.mark.gpu

BAR = 1e-11


def load(name, **kw):
    w = get2d(name).scaled(**kw)
    arr = generate2d(w)
    o = Oracle2D.from_workload(w)
    s = initial_state2d(o, arr)
    ctx = ec.Context2D.from_workload(w)
    ctx.load(arr)
    return w, o, s, ctx


def check(w, g, s):
    for k, L in (("x1", w.L1), ("x2", w.L2)):
        d = np.mod(g[k] - s[k] + L / 2, L) - L / 2
        assert np.abs(d).max() / L < BAR, k
    for k in ("p1", "p2", "e", "bz", "ez", "az") + (("sx", "sy", "sz") if "sx" in s else ()):
        assert np.abs(g[k] - s[k]).max() / np.abs(s[k]).max() < BAR, k


@pytest.mark.parametrize("name,n,sigma,dt", [
    ("twod8x16", 130, 0.1, 0.05),     # few particles a tile, none or one crossing
    ("twod8x16", 512, 0.6, 0.3),      # a row per tile, many crossings in both directions
    ("twod8x16", 513, 0.6, 0.3),
    ("twod16", 4095, 0.8, 0.4),       # about half of the particles cross
    ("twod16s", 2049, 0.6, 0.3),      # with spin
])
def test_rows_of_staying_and_crossing_particles(name, n, sigma, dt):
    """Two Lie steps: the first on the order set_particles makes, the second on the order
    the re-sort makes (expected leavers behind the others)."""
    w, o, s, ctx = load(name, n_particles=n, sigma=sigma, dt=dt)
    with ctx:
        for _ in range(2):
            ctx.step(1)
            st = o.step_s(s, 1)[0] if w.spin != "none" else o.step(s, 1)[0]
            assert st == 0
            check(w, ctx.state(), s)
        assert ctx.gauss_residual() < 1e-12


@pytest.mark.parametrize("name", ["twod16", "twod8x16s"])
def test_substeps_that_need_fewer_sweeps_than_the_last(name):
    """Sweeps store their momentum from the index on at which the last substeps ended; a
    substep that ends earlier (a shorter step, then a still shorter one) commits the same
    momentum as the oracle, and so does the longer one after them."""
    w, o, s, ctx = load(name)
    counts = []
    with ctx:
        for dt in (w.dt, w.dt, w.dt / 8, w.dt / 64, w.dt):
            counts.append(ctx.substep_I(dt)[0])
            r = o.substep_I_s(s, dt) if w.spin != "none" else o.substep_I(s, dt)
            assert r[0] == 0
            check(w, ctx.state(), s)
    assert counts[3] < counts[2] < counts[1] and counts[4] > counts[3], counts


@pytest.mark.parametrize("M1,M2,degree", [(8, 8, 2), (8, 16, 2), (16, 32, 3), (64, 64, 5), (512, 8, 2), (8, 512, 3),
                                          (64, 128, 4), (128, 128, 2)])
def test_solves_keep_the_scheme_on_every_path(M1, M2, degree):
    """The M1 inverse in one block (up to 4096 nodes) or a kernel per direction, with rows
    shorter and longer than the inverse's, and the Subsystem III solve in one block (up
    to 2048) or three kernels, through relations that any solve error breaks: the Gauss
    law after Subsystem I (M1^{-1} of the current) and the energy over Lie steps
    (Subsystem III's matrix as well)."""
    w = get2d("twod16").scaled(L1=M1 * 0.5, L2=M2 * 0.4, M1=M1, M2=M2, degree=degree, n_particles=20 * M1 * M2,
                               dt=0.05, tol=1e-13)
    arr = generate2d(w)
    with ec.Context2D.from_workload(w) as ctx:
        ctx.load(arr)
        H0 = ctx.energy()[5]
        ctx.substep_I()
        # J, M1^{-1} J and the charge are sums of terms of size w to a few 1e-16 relative
        assert ctx.gauss_residual() < 1e-13
        ctx.set_particles(arr["x1"], arr["x2"], arr["p1"], arr["p2"])
        ctx.set_fields(arr["e"], arr["bz"], arr["ez"], arr["az"])
        ctx.solve_gauss()
        ctx.step(3)
        # per step the energy is kept to the fixed points' tolerance (1e-13 absolute per
        # coefficient, against field energies of order 1 per unit area)
        assert abs(ctx.energy()[5] - H0) < 1e-11 * abs(H0)
        assert ctx.gauss_residual() < 1e-13
