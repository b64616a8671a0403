"""GPU tests of the one-launch iterations on frames with defects: dead pixels,
bad columns, borders and sentinels far below the sky, where the smallest value
of a tile's region says nothing about its noise and candidates are held to a
local bound instead; and on dense frames, whose tiles exceed the LDS pool and
list (noise taken for candidates, many cosmic rays).  Bit for bit against the CPU oracle around both tile
shapes, and on large frames no slower than the sparse passes, the general form
(LACOSMIC_FUSED_MAX_PX=0), which do the same work whatever the pixels."""

import numpy as np
import pytest

from gpu_common import assert_bits_equal, host_threads, lac, to_dev

pytestmark = pytest.mark.gpu

F32 = np.float32


def _spoil(img, how):
    g = np.random.Generator(np.random.PCG64(17))
    img = img.copy()
    h, w = img.shape
    if how.startswith("dead"):
        img[g.random(img.shape) < float(how[4:])] = 0.0
    elif how == "column":
        img[:, w // 3] = 0.0
    elif how == "columns":
        img[:, ::16] = 0.0
    elif how == "border":  # rotated onto a larger canvas
        y, x = np.mgrid[0:h, 0:w]
        img[np.abs(y - h / 2) / h + np.abs(x - w / 2) / w > 0.55] = 0.0
    elif how == "frame":  # an overscan's zeros, rows and columns
        img[: h // 8] = img[:, : w // 8] = 0.0
    elif how == "sentinel":
        img[g.random(img.shape) < 1e-3] = F32(-9999.0)
    return img


def _check(img, gain, rn, sigclip=4.5, sepmed=False, u16=False, niter=4, est=False):
    import oracle
    import torch
    L = lac()
    r = oracle.lacosmic(img, gain, rn, sigclip, 0.3, 5.0, niter, nthreads=host_threads(), sepmed=sepmed,
                        estimate_gain=est)
    d = torch.from_numpy(img.astype(np.uint16)).cuda() if u16 else to_dev(img)
    m, c, st = L.run_ex(d, L.make_params(gain, rn, sigclip, 0.3, 5.0, niter, sepmed=sepmed, estimate_gain=est))
    assert_bits_equal(m.cpu().numpy(), r["mask"], "mask")
    assert_bits_equal(c.cpu().numpy(), r["clean"], "clean")
    assert [st.n_new[k] for k in range(niter)] == list(r["n_new"])


# 32 x 32 tiles, and 64 x 64 ones
SHAPES = [(200, 230), (1043, 1051)]
DEFECTS = ["dead1e-3", "dead0.02", "dead0.3", "column", "columns", "border", "frame", "sentinel"]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("how", DEFECTS)
def test_defects_match_the_oracle(how, shape):
    from paper_2602_17938_amd import synth
    p = synth.params_for("cmos")
    img = _spoil(synth.make_frame("cmos", *shape, seed=5), how)
    _check(img, p.gain, p.readnoise, u16=how != "sentinel")


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("sepmed", [False, True])
@pytest.mark.parametrize("how", ["dead0.01", "columns"])
def test_defects_without_read_noise(how, sepmed, shape):
    """Read noise 0: the bound at the smallest value does not apply at all."""
    from paper_2602_17938_amd import synth
    img = _spoil(synth.make_frame("ccd", *shape, seed=6), how)
    _check(img, 1.0, 0.0, sepmed=sepmed)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("case", ["rays", "more rays", "background", "sepmed", "faint", "all", "gain", "estimated",
                                  "negative"])
def test_dense_tiles_match_the_oracle(case, shape):
    """From blocks of S that just exceed the pool (rays) to every pixel of a
    tile evaluated (all)."""
    from paper_2602_17938_amd import synth
    sky = lambda scale=1.0: synth.make_frame("ccd", *shape, seed=8, cr_scale=scale)
    if case == "rays":
        _check(sky(15.0), 1.0, 5.0)
    elif case == "more rays":
        _check(sky(120.0), 1.0, 5.0)
    elif case in ("background", "sepmed"):  # subtracted: the noise model holds the read noise only
        _check((sky() - F32(200.0)).astype(F32), 1.0, 5.0, sepmed=case == "sepmed")
    elif case == "faint":
        _check(sky(), 1.0, 5.0, sigclip=1.0)
    elif case == "all":
        _check(sky(), 1.0, 5.0, sigclip=1e-3, niter=2)
    elif case == "gain":  # five times too large
        p = synth.params_for("cmos")
        _check(synth.make_frame("cmos", *shape, seed=4), 5 * p.gain, p.readnoise, u16=True)
    elif case == "estimated":  # (the estimate's bins lie in the plane that holds a dense tile's S)
        _check(sky(30.0), 0.0, 5.0, sigclip=1.5, est=True, niter=3)
    else:
        _check((sky() * F32(-1.0)).astype(F32), 1.0, 5.0, sigclip=2.0)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("side,step", [(26, 1), (56, 3)])
def test_more_pixels_to_evaluate_than_the_list_holds(side, step, shape):
    """Bright pixels and a sigfrac so small that nearly every pixel beside one is
    evaluated, on 64 x 64 tiles more of them than the list holds while the
    candidates still fit it: 26 x 26 pixels side by side (390 candidates, 256
    blocks: all the pool holds, 536 pixels of 512), and every third of 56 x 56
    (380, 1296, 2358 pixels of 2048)."""
    import oracle
    L = lac()
    h, w = shape
    g = np.random.Generator(np.random.PCG64(41))
    img = g.poisson(200.0, size=shape) + g.normal(0, 5.0, size=shape)
    for y0 in range(7, h - side, 64):
        for x0 in range(5, w - side, 64):
            img[y0:y0 + side:step, x0:x0 + side:step] += g.uniform(2000, 20000, (-(-side // step),) * 2)
    img = img.astype(F32)
    r = oracle.lacosmic(img, 1.0, 5.0, 8.0, 1e-4, 0.01, 4, nthreads=host_threads())
    for _ in range(5):
        m, c, st = L.run_ex(to_dev(img), L.make_params(1.0, 5.0, 8.0, 1e-4, 0.01, 4))
        assert_bits_equal(m.cpu().numpy(), r["mask"], "mask")
        assert_bits_equal(c.cpu().numpy(), r["clean"], "clean")
        assert [st.n_new[k] for k in range(4)] == list(r["n_new"])


def test_dense_frames_in_a_batch():
    from paper_2602_17938_amd import synth
    L = lac()
    imgs = [synth.make_frame("ccd", 700, 811, seed=3), synth.make_frame("ccd", 900, 640, seed=4, cr_scale=60.0)]
    imgs.append((imgs[0][:500] - F32(200.0)).astype(F32))
    masks, cleans = L.run_batch([to_dev(x) for x in imgs], L.make_params(1.0, 5.0, 2.0, 0.3, 5.0, 4))
    for i, img in enumerate(imgs):
        import oracle
        r = oracle.lacosmic(img, 1.0, 5.0, 2.0, 0.3, 5.0, 4, nthreads=host_threads())
        assert_bits_equal(masks[i].cpu().numpy(), r["mask"], "mask %d" % i)
        assert_bits_equal(cleans[i].cpu().numpy(), r["clean"], "clean %d" % i)


@pytest.mark.parametrize("shape", SHAPES)
def test_nonfinite_pixels_in_dense_tiles(shape):
    from paper_2602_17938_amd import synth
    L = lac()
    img = (synth.make_frame("ccd", *shape, seed=8) - F32(200.0)).astype(F32)
    for bad in (np.nan, np.inf, -np.inf):
        x = img.copy()
        x[shape[0] // 2, shape[1] // 3] = bad
        with pytest.raises(L.LacosmicError) as e:
            L.run_ex(to_dev(x), L.make_params(1.0, 5.0, 0.5))
        assert e.value.status == L.ENONFINITE


def _ms(call):
    import torch
    best = 1e9
    for _ in range(6):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(4):
            call()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 4)
    return best


def _tiles_against_passes(img, gain, rn, sigclip, monkeypatch):
    import torch
    L = lac()
    p = L.make_params(gain, rn, sigclip, 0.3, 5.0, 4)
    m = torch.zeros(img.shape, dtype=torch.uint8, device="cuda")
    c = torch.zeros(img.shape, dtype=torch.float32, device="cuda")
    call = lambda: L.run_ex(img, p, m, c, stats=False)
    call()
    tiles = _ms(call)
    got = m.clone(), c.clone()
    monkeypatch.setenv("LACOSMIC_FUSED_MAX_PX", "0")
    call()
    passes = _ms(call)
    assert torch.equal(got[0], m) and torch.equal(got[1].view(torch.int32), c.view(torch.int32))
    print("tiles %.3f ms, passes %.3f ms" % (tiles, passes), flush=True)
    return tiles / passes


def _large(kind, how, copies=4):
    """Copies of a spoilt frame side by side, as the camera delivers it."""
    import torch
    from paper_2602_17938_amd import synth
    shape = (1024, 1024) if kind == "ccd" else (1600, 2400)
    x = torch.from_numpy(_spoil(synth.make_frame(kind, *shape, seed=9), how)).cuda().repeat(copies, copies)
    return x.to(torch.int32).to(torch.uint16) if kind == "cmos" else x.contiguous()


# Run to run both forms vary by a few percent; a bound that fails on a defect
# makes the tiles 1.5 to 3 times as slow as the passes.
LIMIT = 1.25


@pytest.mark.parametrize("kind,how,rn", [("ccd", "none", None), ("cmos", "none", None), ("ccd", "dead1e-3", None),
                                         ("ccd", "dead1e-3", 0.0), ("cmos", "dead1e-4", None),
                                         ("cmos", "dead1e-3", None), ("cmos", "dead1e-3", 0.0),
                                         ("cmos", "column", None), ("cmos", "border", None)])
def test_defects_do_not_slow_the_tiles(kind, how, rn, monkeypatch):
    from paper_2602_17938_amd import synth
    p = synth.params_for(kind)
    ratio = _tiles_against_passes(_large(kind, how), p.gain, p.readnoise if rn is None else rn, 4.5, monkeypatch)
    assert ratio < LIMIT


@pytest.mark.parametrize("kind,sigclip,sky", [("ccd", 4.5, 200.0), ("cmos", 4.5, 200.0), ("ccd", 2.0, 0.0),
                                              ("ccd", 1.0, 0.0), ("cmos", 1.0, 0.0)])
def test_dense_frames_do_not_slow_the_tiles(kind, sigclip, sky, monkeypatch):
    """A background (sky) subtracted, or a low detection limit."""
    import torch
    from paper_2602_17938_amd import synth
    p = synth.params_for(kind)
    x = _large(kind, "none")
    if sky:
        x = x.to(torch.int32).to(torch.float32) - sky if kind == "cmos" else x - sky
    assert _tiles_against_passes(x, p.gain, p.readnoise, sigclip, monkeypatch) < LIMIT


def test_defects_do_not_slow_the_largest_frames(monkeypatch):
    """Far above the size up to which frames run on tiles, whose time per pixel
    grows with the defects where the passes' does not."""
    from paper_2602_17938_amd import synth
    p = synth.params_for("cmos")
    x = _large("cmos", "dead1e-3", 12)  # 553 Mpx
    assert _tiles_against_passes(x, p.gain, p.readnoise, 4.5, monkeypatch) < 1.15
    lac().shutdown()  # (its workspace: 9 GB)
