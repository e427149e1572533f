"""Large readouts go through a pinned ring: 2 MiB slots, 16 of them, from 8 MiB up.

Tolerance: momenta and spins are stored and returned as given, so they are equal bit by
bit; positions pass through cell units (one product each way), hence a few ulp of L.
"""
import numpy as np
import pytest

import paper_2203_06513_amd as ec
from workloads.twod import get2d

pytestmark = pytest.mark.gpu

SLOT = 2 << 17                 # doubles of a 2 MiB slot
SIZES = [4 * SLOT - 1,         # below the ring's smallest size: the plain copy
         4 * SLOT,             # whole slots only
         4 * SLOT + 1,         # a last slot of one value
         16 * SLOT,            # each slot once
         35 * SLOT + 77]       # slots filled again


@pytest.mark.parametrize("n", SIZES)
def test_1d_round_trip(n):
    rng = np.random.default_rng(n)
    L = 8.0
    ctx = ec.Context(L=L, M=64, degree=3, n_particles=n, dt=0.01, tol=1e-12, spin=True, hbar=0.01)
    x, p = rng.uniform(0, 0.999 * L, n), rng.normal(size=n)
    s = [rng.normal(size=n) for _ in range(3)]
    ctx.set_particles(x, p)
    ctx.set_spins(*s)
    for _ in range(2):
        gx, gp = ctx.get_particles()
        assert np.array_equal(gp, p)
        assert np.abs(gx - x).max() <= 4 * np.finfo(float).eps * L
        for a, b in zip(ctx.get_spins(), s):
            assert np.array_equal(a, b)
    ctx.close()


@pytest.mark.parametrize("n", SIZES)
def test_2d_round_trip(n):
    rng = np.random.default_rng(n)
    w = get2d("twod16s").scaled(n_particles=n)
    ctx = ec.Context2D.from_workload(w)
    x = [rng.uniform(0, 0.999 * L, n) for L in (w.L1, w.L2)]
    p = [rng.normal(size=n) for _ in range(2)]
    s = [rng.normal(size=n) for _ in range(3)]
    ctx.set_particles(*x, *p)
    ctx.set_spins(*s)
    g = ctx.get_particles()
    for k, v, L in (("x1", x[0], w.L1), ("x2", x[1], w.L2)):
        assert np.abs(g[k] - v).max() <= 4 * np.finfo(float).eps * L
    assert np.array_equal(g["p1"], p[0]) and np.array_equal(g["p2"], p[1])
    gs = ctx.get_spins()
    for k, v in zip(("sx", "sy", "sz"), s):
        assert np.array_equal(gs[k], v)
    ctx.close()
