"""A readout waits for its context's own stream only: field readouts into pinned and into
device memory return while work of another stream (0.3 s and more of matrix products) is
still running.  Streams share a few hardware queues, and one that shares the other's has to
wait for it; of eight streams at least one does not, and a readout that waits for other
streams waits on all of them."""
import numpy as np
import pytest

import paper_2203_06513_amd as ec
from paper_2203_06513_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["pageable", "pinned", "device"])
def test_field_readout_does_not_wait_for_other_streams(where):
    torch = pytest.importorskip("torch")
    M = 16
    rng = np.random.default_rng(1)
    f = {k: rng.normal(size=M) for k in ("ex", "ey", "ez", "ay", "az")}
    a = torch.rand(8192, 8192, device="cuda")
    b = a.mm(a)
    kw = dict(pageable={}, pinned=dict(pin_memory=True), device=dict(device="cuda"))[where]
    waited = []
    for _ in range(8):
        own = torch.cuda.Stream()
        out = [torch.zeros(M, dtype=torch.float64, **kw) for _ in f]
        with ec.Context(8.0, M, 3, 0, 0.01, 1e-12, stream=own.cuda_stream) as c:
            c.set_fields(**f)
            torch.cuda.synchronize()
            for _ in range(40):
                torch.mm(a, a, out=b)
            end = torch.cuda.Event()
            end.record()
            assert _lib.load().ecpic_get_fields(c._h, *[v.data_ptr() for v in out]) == 0
            waited.append(end.query())
        torch.cuda.synchronize()
        for v, w in zip(out, f.values()):
            assert np.array_equal(v.cpu().numpy(), w)
        if not waited[-1]:
            break
    assert not all(waited)
