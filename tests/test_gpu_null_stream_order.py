"""GPU tests of the order between the legacy null stream and calls that name no
stream: kernels enqueued there just before the call -- writing its input, the
workspace that holds its frame record, its outputs -- come first, whether they
still run when the call is made or have just ended."""

import numpy as np
import pytest

from gpu_common import lac, to_dev

pytestmark = pytest.mark.gpu

F32 = np.float32


@pytest.mark.parametrize("entry", ["run", "run_ex", "workspace", "batch"])
@pytest.mark.parametrize("pause", [0.0, 2e-5, 2e-4])
def test_calls_come_after_the_null_streams_kernels(entry, pause):
    import time
    import torch
    from paper_2602_17938_amd import synth
    L = lac()
    h, w = 210, 333
    imgs = [to_dev(synth.make_frame("ccd", h, w, seed=s)) for s in (1, 2)]
    p = L.make_params(1.0, 5.0)
    want = [L.run_ex(x, p)[:2] for x in imgs]
    assert not torch.equal(want[0][0], want[1][0])
    x = imgs[0].clone()
    m = torch.zeros((h, w), dtype=torch.uint8, device="cuda")
    c = torch.zeros((h, w), dtype=torch.float32, device="cuda")
    ws = L.alloc_workspace(h, w)
    for k in range(60):
        x.copy_(imgs[k % 2])
        m.fill_(7)
        c.fill_(-1.0)
        ws.fill_(0xA5)
        if pause:
            time.sleep(pause)
        if entry == "run":
            got = L.run(x, 1.0, 5.0)
        elif entry == "run_ex":
            got = L.run_ex(x, p, m, c, stream=None)[:2]
        elif entry == "workspace":
            got = L.run_ex(x, p, m, c, workspace=ws, stream=None)[:2]
        else:
            got = [t[0] for t in L.run_batch([x], p, [m], [c], stream=None)]
        assert torch.equal(got[0], want[k % 2][0]), "call %d mask" % k
        assert torch.equal(got[1], want[k % 2][1]), "call %d clean" % k
