"""Steps on grids up to and past 128 cells, where the field updates open the sweeps and
commits instead of running as kernels of their own: every degree, one to four waves a cell,
empty cells, cells of several work items, fewer cells than taps, with and without spin,
against the oracle.

Tolerance: both sides stop their fixed points at 1e-13 on the same maps, whose contraction
here is below 1/2, so a step leaves states a few 1e-13 apart; three steps of states of order
1, hence 1e-11, the bar of the other parity tests of whole steps.
"""
import numpy as np
import pytest

import paper_2203_06513_amd as ec
import workloads
from oracle import Oracle, initial_state

pytestmark = pytest.mark.gpu

BAR = 1e-11


def run(w, arr, steps=3, seidel=1, splitting=0, **kw):
    o = Oracle.from_workload(w, seidel=seidel, splitting=splitting)
    s = initial_state(o, arr)
    start = dict(arr, ex=s["ex"].copy())
    assert o.step(s, steps)[0] == 0
    with ec.Context.from_workload(w, map=ec.MAP_SEIDEL if seidel else ec.MAP_JACOBI, splitting=splitting, **kw) as c:
        c.load(start, solve_gauss=False)
        rc, done, *_ = c.step(steps)
        g = c.state()
    assert rc == 0 and done == steps
    for k in g:
        d = np.asarray(g[k]) - np.asarray(s[k])
        if k == "x":
            d = np.mod(d + w.L / 2, w.L) - w.L / 2
        assert np.abs(d).max() <= BAR * max(1.0, np.abs(s[k]).max()), k


@pytest.mark.parametrize("seidel", [0, 1])
@pytest.mark.parametrize("degree", [2, 3, 4, 5])
@pytest.mark.parametrize("M", [8, 63, 64, 65, 127, 128, 129])
def test_cells(M, degree, seidel):
    w = workloads.get("paper51").scaled(degree=degree, M=M, n_particles=3001)
    run(w, workloads.generate(w), seidel=seidel)


@pytest.mark.parametrize("splitting", [0, 1])
@pytest.mark.parametrize("wpi", [1, 2, 3, 4])
@pytest.mark.parametrize("spin", [False, True])
def test_waves(spin, wpi, splitting):
    w = workloads.get("paper52" if spin else "paper51").scaled(M=32, n_particles=6000)
    run(w, workloads.generate(w), splitting=splitting, waves_per_item=wpi)


@pytest.mark.parametrize("splitting", [0, 1])
@pytest.mark.parametrize("degree", [2, 5])
@pytest.mark.parametrize("n", [1, 2, 40])
def test_empty_cells(n, degree, splitting):
    w = workloads.get("paper51").scaled(degree=degree, M=64, n_particles=n)
    run(w, workloads.generate(w), splitting=splitting)


@pytest.mark.parametrize("splitting", [0, 1])
@pytest.mark.parametrize("degree", [3, 4])
def test_cells_of_several_items(degree, splitting):
    """1875 particles a cell in the mean, up to 2200 with the ripple, items of 2048."""
    w = workloads.get("paper51").scaled(degree=degree, M=16, n_particles=30000)
    arr = dict(workloads.generate(w))
    x = arr["x"]
    arr["x"] = np.mod(x + 0.2 * w.L / (2 * np.pi) * np.sin(2 * np.pi * x / w.L), w.L)
    assert np.bincount((arr["x"] / (w.L / 16)).astype(int), minlength=16).max() > 2100
    run(w, arr, splitting=splitting, item_particles=2048)
