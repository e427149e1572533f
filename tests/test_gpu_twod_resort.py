"""The 2D re-sort of tiles around and past the 6144 particles that pass through LDS (a
fuller tile writes each particle to its place directly): every particle is there once.

With a weight of 1e-40 the fields stay below 1e-30, so Subsystem I leaves momenta and (with
hbar = 0) spins bit by bit as they were, in the caller's order; a particle lost or written
twice leaves another one's value, or none, in its place.  Positions advance by
dt p / sqrt(1 + p^2) a substep: three roundings a step and one product each way, 1e-14 of L.
"""
import numpy as np
import pytest

import paper_2203_06513_amd as ec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["row", "column0", "all"])
@pytest.mark.parametrize("n", [6143, 6144, 6145, 12000, 60000])
def test_every_particle_is_there_once(n, where):
    rng = np.random.default_rng(n)
    M, dt, steps = 8, 0.2, 4
    L = 0.5 * M
    x1, x2 = rng.uniform(0, L, n), rng.uniform(0, L, n)
    if where == "row":          # one tile holds all of them at first
        x1 = rng.uniform(1.0, 1.49, n)
    elif where == "column0":    # and they share two sort keys: column 0, expected to stay or to leave
        x1, x2 = rng.uniform(1.0, 1.49, n), rng.uniform(0, 0.49, n)
    p = [rng.normal(size=n) for _ in range(2)]
    s = [rng.normal(size=n) for _ in range(3)]
    g = np.sqrt(1.0 + p[0] ** 2 + p[1] ** 2)
    with ec.Context2D(L, L, M, M, 2, n, dt, 1e-13, weight=1e-40, spin=1) as c:
        c.set_particles(x1, x2, *p)
        c.set_spins(*s)
        for k in range(1, steps + 1):
            c.substep_I()
            q = c.get_particles()
            for a, b in zip((q["p1"], q["p2"], *c.get_spins().values()), (*p, *s)):
                assert np.array_equal(a, b)
            for a, b, v in ((q["x1"], x1, p[0]), (q["x2"], x2, p[1])):
                d = a - (b + k * dt * v / g)
                assert np.abs(np.mod(d + L / 2, L) - L / 2).max() <= 1e-14 * L * k
