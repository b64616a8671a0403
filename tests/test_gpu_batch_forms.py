"""GPU tests of lacosmic_run_batch's forms and arguments: what the binding
accepts, tables of many frames, and the launches per pass (with their recorded
graph), which batches of ordinary test sizes do not run by themselves."""

import numpy as np
import pytest

from gpu_common import assert_bits_equal, host_threads, lac, to_dev

pytestmark = pytest.mark.gpu

F32 = np.float32


def _oracle(img, p, **kw):
    import oracle
    return oracle.lacosmic(img, p.gain, p.readnoise, p.sigclip, p.sigfrac, p.objlim, p.niter,
                           nthreads=host_threads(), **kw)


def test_parameters_and_outputs_from_any_iterable():
    import torch
    from paper_2602_17938_amd import synth
    L = lac()
    p = synth.params_for("ccd")
    q = L.make_params(p.gain, p.readnoise, p.sigclip, p.sigfrac, p.objlim, p.niter)
    imgs = [synth.make_frame("ccd", 90 + 5 * k, 110, seed=k) for k in range(3)]
    dev = [to_dev(x) for x in imgs]
    masks = [torch.zeros(x.shape, dtype=torch.uint8, device="cuda") for x in dev]
    cleans = {k: torch.zeros(x.shape, dtype=torch.float32, device="cuda") for k, x in enumerate(dev)}
    L.run_batch(dev, (q for _ in range(3)), (m for m in masks), cleans.values())
    L.run_batch(tuple(dev), {k: q for k in range(4)}.values(), masks, iter(cleans.values()))
    torch.cuda.synchronize()
    for k, img in enumerate(imgs):
        r = _oracle(img, p)
        assert_bits_equal(masks[k].cpu().numpy(), r["mask"], "mask %d" % k)
        assert_bits_equal(cleans[k].cpu().numpy(), r["clean"], "clean %d" % k)
    with pytest.raises(IndexError):
        L.run_batch(dev[:2], q, (m for m in masks), list(cleans.values())[:2])
