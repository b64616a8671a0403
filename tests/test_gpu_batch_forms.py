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


# --------------------------------------------------------- tables of many frames
@pytest.mark.parametrize("n", [65, 200])
@pytest.mark.parametrize("edge", [40, 130])
def test_tables_of_more_frames_than_a_wave(n, edge):
    """A tile's frame is found by narrowing the table 64-fold; frames of one to
    nine tiles, and iterations that run listed tiles only."""
    import torch
    from paper_2602_17938_amd import synth
    L = lac()
    p = synth.params_for("ccd")
    g = np.random.Generator(np.random.PCG64(n + edge))
    base = synth.make_frame("ccd", 400, 400, seed=edge, cr_scale=4.0)
    imgs = []
    for _ in range(n):
        h, w = (int(v) for v in g.integers(1, edge, 2))
        y, x = int(g.integers(0, 400 - h)), int(g.integers(0, 400 - w))
        imgs.append(np.ascontiguousarray(base[y:y + h, x:x + w]))
    q = L.make_params(p.gain, p.readnoise, p.sigclip, p.sigfrac, p.objlim, 5)
    masks, cleans = L.run_batch([to_dev(x) for x in imgs], q)
    torch.cuda.synchronize()
    import oracle
    flagged = 0
    for k, img in enumerate(imgs):
        r = oracle.lacosmic(img, p.gain, p.readnoise, p.sigclip, p.sigfrac, p.objlim, 5)
        flagged += int(r["mask"].sum())
        assert_bits_equal(masks[k].cpu().numpy(), r["mask"], "mask %d" % k)
        assert_bits_equal(cleans[k].cpu().numpy(), r["clean"], "clean %d" % k)
    assert flagged > 50


# ------------------------------------------------------------- launches per pass
# LACOSMIC_BATCH_PLAN: tile shape, launch form (0 queue, 1 grid), groups.
PLANS = ["1,1,1", "1,1,3", "0,1,2", "2,0,2"]


@pytest.fixture(params=PLANS)
def plan(request, monkeypatch):
    monkeypatch.setenv("LACOSMIC_BATCH_PLAN", request.param)
    return request.param


# A plan is kept for the last batch shape only: each case adds its own frame.
def _frames(case, plan, specs, seed=0):
    from paper_2602_17938_amd import synth
    salt = (sorted(["options", "replay", "early", "streams", "wide", "bad"]).index(case), PLANS.index(plan))
    specs = list(specs) + [("ccd", 20 + 3 * salt[0], 31 + 2 * salt[1])]
    return specs, [synth.make_frame(k, h, w, seed=seed + 7 * j) for j, (k, h, w) in enumerate(specs)]


def _ran(plan):
    L = lac().lib()
    cfg, mode, groups = (int(v) for v in plan.split(","))
    assert (L.lacosmic_batch_tile_shape(), L.lacosmic_batch_launch_mode(), L.lacosmic_batch_groups()) == (cfg, mode, groups)


RAGGED = [("ccd", 517, 333), ("cmos", 200, 650), ("ccd", 1, 77), ("cmos", 129, 64), ("ccd", 65, 1)]


def _batch(imgs, params, **kw):
    """The batch's results as host arrays, its inputs of uint16 where the
    parameters say so."""
    import torch
    L = lac()
    dev = [torch.from_numpy(x.astype(np.uint16)).cuda() if u else to_dev(x) for x, (_, u) in zip(imgs, params)]
    masks, cleans = L.run_batch(dev, [q for q, _ in params], **kw)
    torch.cuda.synchronize()
    return [m.cpu().numpy() for m in masks], [c.cpu().numpy() for c in cleans]


def test_passes_with_options_replayed(plan):
    """Estimated gain, separable medians, uint16 input and other gains side by
    side, and the recorded graph replayed with other images, parameters and
    buffers (and other work of the program in between)."""
    import torch
    from paper_2602_17938_amd import synth
    L = lac()
    for rep in range(3):
        specs, imgs = _frames("options", plan, RAGGED, seed=100 * rep)
        params, want = [], []
        for j, ((kind, _, _), img) in enumerate(zip(specs, imgs)):
            p = synth.params_for(kind)
            est, sep, u16 = (j + rep) % 4 == 0, (j + rep) % 3 == 0, kind == "cmos"
            gain = p.gain * (1.7 if (j + rep) % 2 else 1.0)
            params.append((L.make_params(0.0 if est else gain, p.readnoise, 4.5, 0.3, 5.0 - rep, 4,
                                         estimate_gain=est, sepmed=sep), u16))
            q = synth.FrameParams(gain=0.0 if est else gain, readnoise=p.readnoise, objlim=5.0 - rep, niter=4)
            want.append(_oracle(img, q, estimate_gain=est, sepmed=sep))
        masks, cleans = _batch(imgs, params)
        _ran(plan)
        for k, r in enumerate(want):
            assert_bits_equal(masks[k], r["mask"], "rep %d mask %d" % (rep, k))
            assert_bits_equal(cleans[k], r["clean"], "rep %d clean %d" % (rep, k))
        torch.randn(1 << 20, device="cuda").sum().item()


def test_passes_early_stop_replayed(plan):
    from paper_2602_17938_amd import synth
    L = lac()
    for rep in range(3):
        specs, imgs = _frames("early", plan, RAGGED, seed=50 * rep)
        ps = [synth.params_for(k) for k, _, _ in specs]
        params = [(L.make_params(p.gain, p.readnoise, niter=8, early_stop=True), False) for p in ps]
        masks, cleans = _batch(imgs, params)
        _ran(plan)
        for k, (img, p) in enumerate(zip(imgs, ps)):
            r = _oracle(img, synth.FrameParams(gain=p.gain, readnoise=p.readnoise, niter=8), early_stop=True)
            assert_bits_equal(masks[k], r["mask"], "rep %d mask %d" % (rep, k))
            assert_bits_equal(cleans[k], r["clean"], "rep %d clean %d" % (rep, k))


def test_passes_on_two_streams(plan):
    """Two asynchronous calls share the plan, its frame table and workspaces."""
    import torch
    from paper_2602_17938_amd import synth
    L = lac()
    sets = [_frames("streams", plan, RAGGED[:3], seed=30 * s) for s in range(2)]
    params = [L.make_params(synth.params_for(k).gain, synth.params_for(k).readnoise) for k, _, _ in sets[0][0]]
    L.run_batch([to_dev(x) for x in sets[0][1]], params)
    _ran(plan)
    dev = [[to_dev(x) for x in imgs] for _, imgs in sets]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [L.run_batch(dev[s], params, stream=streams[s]) for s in range(2)]
    for s in streams:
        s.synchronize()
    for s in range(2):
        for k, ((kind, _, _), img) in enumerate(zip(*sets[s])):
            r = _oracle(img, synth.params_for(kind))
            assert_bits_equal(outs[s][0][k].cpu().numpy(), r["mask"], "stream %d mask %d" % (s, k))
            assert_bits_equal(outs[s][1][k].cpu().numpy(), r["clean"], "stream %d clean %d" % (s, k))


def test_passes_on_wide_rows(plan):
    """Rows of one and of two strip columns."""
    from paper_2602_17938_amd import synth
    specs, imgs = _frames("wide", plan, [("ccd", 37, 4032), ("ccd", 35, 4097), ("ccd", 18, 8000)])
    p = synth.params_for("ccd")
    q = lac().make_params(p.gain, p.readnoise)
    masks, cleans = _batch(imgs, [(q, False)] * len(imgs))
    _ran(plan)
    for k, img in enumerate(imgs):
        r = _oracle(img, p)
        assert_bits_equal(masks[k], r["mask"], "mask %d" % k)
        assert_bits_equal(cleans[k], r["clean"], "clean %d" % k)


def test_passes_report_a_nonfinite_frame(plan):
    L = lac()
    _, imgs = _frames("bad", plan, RAGGED[:2])
    imgs[1][100, 300] = np.nan
    with pytest.raises(L.LacosmicError) as e:
        L.run_batch([to_dev(x) for x in imgs], L.make_params(1.0, 5.0), stream=None)
    assert e.value.status == L.ENONFINITE
    _ran(plan)
    imgs[1][100, 300] = 200.0  # the plan replayed
    L.run_batch([to_dev(x) for x in imgs], L.make_params(1.0, 5.0), stream=None)
