"""Steps queued behind each other are joined by one kernel, of two blocks from 65 cells on;
up to 128 cells each of them reads the whole constant part of the Subsystem II iteration
and forms its cells of the next step's.  A batch of steps is therefore the same steps one
call at a time (which no kernel joins), bit for bit, also when the blocks of a launch do not
start together because other streams keep the GPU busy.
"""
import numpy as np
import pytest

import paper_2203_06513_amd as ec
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spin", [False, True])
@pytest.mark.parametrize("M,degree", [(64, 3), (65, 2), (96, 5), (127, 4), (128, 3), (129, 3), (200, 5)])
def test_batches_are_their_steps(M, degree, spin):
    torch = pytest.importorskip("torch")
    w = workloads.get("paper52" if spin else "paper51").scaled(M=M, degree=degree, n_particles=3000)
    arr = workloads.generate(w)
    side = [torch.cuda.Stream() for _ in range(3)]
    a = torch.rand(1024, 1024, device="cuda")
    out = []
    for calls in ([16, 13], [1] * 29):
        with ec.Context.from_workload(w, map=ec.MAP_SEIDEL) as c:
            c.load(arr)
            for n in calls:
                if n > 1:
                    for s in side:
                        with torch.cuda.stream(s):
                            for _ in range(20):
                                a.mm(a)
                rc, done, *_ = c.step(n)
                assert rc == 0 and done == n
            torch.cuda.synchronize()
            out.append(c.state())
    for k in out[0]:
        np.testing.assert_array_equal(out[0][k], out[1][k], err_msg=k)
