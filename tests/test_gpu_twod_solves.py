"""The M1 inverse in its two kernels on the shapes where they differ: row blocks of fewer than
64 rows (and the last block of columns partly past the grid), and quintic rows of 205 entries
on 256 rows and more (66 KB and more of LDS a block).

By relations that any solve error breaks: the Gauss law after Subsystem I (J, M1^{-1} J and the
charge are sums of terms of size w to a few 1e-16 relative), and the energy over Lie steps,
kept to the fixed points' tolerance of 1e-13 absolute per coefficient, against field energies
of order 1 per unit area.
"""
import pytest

import paper_2203_06513_amd as ec
from workloads.twod import generate2d, get2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M1,M2,degree", [(16, 512, 3), (16, 512, 5), (32, 256, 4), (512, 16, 3),
                                          (512, 16, 5), (256, 32, 5), (256, 256, 5)])
def test_two_kernel_solves_keep_the_scheme(M1, M2, degree):
    n = min(20 * M1 * M2, 400_000)
    w = get2d("twod16").scaled(L1=M1 * 0.5, L2=M2 * 0.4, M1=M1, M2=M2, degree=degree, n_particles=n, dt=0.05,
                               tol=1e-13)
    arr = generate2d(w)
    with ec.Context2D.from_workload(w) as ctx:
        ctx.load(arr)
        H0 = ctx.energy()[5]
        ctx.substep_I()
        assert ctx.gauss_residual() < 1e-13
        ctx.set_particles(arr["x1"], arr["x2"], arr["p1"], arr["p2"])
        ctx.set_fields(arr["e"], arr["bz"], arr["ez"], arr["az"])
        ctx.solve_gauss()
        ctx.step(3)
        assert abs(ctx.energy()[5] - H0) < 1e-11 * abs(H0)
        assert ctx.gauss_residual() < 1e-13
