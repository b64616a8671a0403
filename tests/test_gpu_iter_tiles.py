"""GPU parity of the one-launch iterations (lacosmic_iter.h) where they can go
wrong: frame sizes around the tile sizes (32 and 64 pixels, with partial tiles
and frames narrower than a tile), tiles too dense for one pass over their
candidates, values on both sides of zero, objlim decisions near and far from
the bound, integer-valued frames (ties everywhere), the estimated gain (every
tile active in every iteration), uint16 input, and iterations that skip most
tiles.  Everything against the CPU oracle, bit for bit."""

import numpy as np
import pytest

from gpu_common import assert_bits_equal, host_threads, lac, to_dev

pytestmark = pytest.mark.gpu

F32 = np.float32


def _sky(h, w, seed, level=200.0, density=1.0 / 60, scale=1.0):
    """Poisson sky, a few stars, and single hot pixels and short tracks on a
    fraction of the pixels, the borders included."""
    g = np.random.Generator(np.random.PCG64(seed))
    img = g.poisson(level, size=(h, w)) + g.normal(0, 5.0, size=(h, w))
    for _ in range(max(1, h * w // 9000)):
        y0, x0, s = g.uniform(0, h), g.uniform(0, w), g.uniform(1.1, 1.7)
        ya, yb, xa, xb = max(0, int(y0) - 8), min(h, int(y0) + 9), max(0, int(x0) - 8), min(w, int(x0) + 9)
        yy, xx = np.mgrid[ya:yb, xa:xb]
        img[ya:yb, xa:xb] += g.uniform(500, 30000) * np.exp(-((yy - y0) ** 2 + (xx - x0) ** 2) / (2 * s * s))
    n = max(2, int(h * w * density))
    ys, xs = g.integers(0, h, n), g.integers(0, w, n)
    img[ys, xs] += g.uniform(100, 20000, n)
    k = ys < h - 1
    img[ys[k][::3] + 1, xs[k][::3]] += 900.0
    img[0, 0] += 5000
    img[h - 1, w - 1] += 4000
    return (img * scale).astype(F32)


def _check(img, gain=1.0, rn=5.0, sigclip=4.5, sigfrac=0.3, objlim=5.0, niter=5, early=False,
           est=False, sepmed=False, u16=False, flags=True):
    import oracle
    import torch
    L = lac()
    r = oracle.lacosmic(img, 0.0 if est else gain, rn, sigclip, sigfrac, objlim, niter,
                        early_stop=early, nthreads=host_threads(), estimate_gain=est, sepmed=sepmed)
    p = L.make_params(0.0 if est else gain, rn, sigclip, sigfrac, objlim, niter, early,
                      estimate_gain=est, sepmed=sepmed)
    d = torch.from_numpy(img.astype(np.uint16)).cuda() if u16 else to_dev(img)
    m, c, st = L.run_ex(d, p)
    assert_bits_equal(m.cpu().numpy(), r["mask"], "mask")
    assert_bits_equal(c.cpu().numpy(), r["clean"], "clean")
    n = st.iters_run
    assert [st.n_new[k] for k in range(n)] == list(r["n_new"])[:n]
    assert st.n_unreplaced == r["n_unreplaced"]
    assert not flags or int(r["mask"].sum()) > 0  # the inputs are meant to have cosmic rays


# small tiles: below 2^20 pixels; the last three run 64 x 64 tiles
SIZES = [(31, 33), (32, 64), (65, 31), (48, 48), (80, 81), (97, 16), (8, 200), (257, 129),
         (1025, 1024), (1087, 1029), (640, 1729)]


@pytest.mark.parametrize("shape", SIZES)
def test_sizes_around_the_tiles(shape):
    _check(_sky(*shape, seed=shape[0] * 31 + shape[1]))


@pytest.mark.parametrize("shape,density", [((200, 210), 0.08), ((200, 210), 0.3), ((1100, 1000), 0.06),
                                           ((1100, 1000), 0.25)])
def test_dense_tiles(shape, density):
    _check(_sky(*shape, seed=7, density=density), niter=4)


@pytest.mark.parametrize("shape", [(150, 170), (1030, 1040)])
@pytest.mark.parametrize("case", ["negative", "integer", "faint", "gain", "sepmed", "est", "u16", "low"])
def test_values_and_options(shape, case):
    img = _sky(*shape, seed=len(case) * 7 + shape[0])
    if case == "negative":  # background-subtracted: the keys of negative values
        _check((img - F32(200.0)).astype(F32))
    elif case == "integer":
        _check(np.rint(img / 8).astype(F32), gain=2.0)
    elif case == "faint":  # the objlim ratio near its limit for many pixels
        g = np.random.Generator(np.random.PCG64(3))
        _check((img + g.uniform(0, 90, img.shape)).astype(F32), objlim=1.2, sigclip=3.0)
    elif case == "gain":
        _check(img, gain=1.7, rn=3.3, niter=4)
    elif case == "sepmed":
        _check(img, sepmed=True)
    elif case == "est":
        _check(img, est=True, niter=3)
    elif case == "u16":
        _check(np.clip(np.rint(img), 0, 65535).astype(F32), u16=True, early=True, niter=8)
    else:  # nearly every pixel is a candidate, and growth goes far
        _check(img, sigclip=0.5, sigfrac=0.5, objlim=0.5, niter=3)


def test_values_where_the_bounds_overflow():
    """Values up to 2^100 (the candidates' bound does not apply) and a tiny
    gain and sigclip: every pixel takes the exact path."""
    img = _sky(90, 100, seed=5)
    big = img.copy()
    big[30:60, 20:70] *= F32(2.0 ** 95)
    _check(big)
    _check(img, gain=2.0 ** -40, niter=2, flags=False)  # the read noise covers everything
    _check((img * F32(2.0 ** 40)).astype(F32), gain=2.0 ** -40, niter=2)
    _check((img * F32(1e-30)).astype(F32), gain=1.0, rn=0.0, niter=2, flags=False)  # all below the floor


@pytest.mark.parametrize("sepmed", [False, True])
@pytest.mark.parametrize("shape,most", [((512, 544), 60), ((1088, 1024), 110)])
def test_tiles_of_every_load(shape, most, sepmed):
    # from tile to tile, 0 .. most isolated bright pixels, and star cores of as
    # many rejected pixels: all block counts from none to past the pool, a few
    # and many candidates whose objlim test is close
    h, w = shape
    g = np.random.Generator(np.random.PCG64(99))
    img = g.poisson(200.0, size=shape) + g.normal(0, 5.0, size=shape)
    e = 32 if h * w <= 1 << 20 else 64
    for k, (y, x) in enumerate((y, x) for y in range(0, h, e) for x in range(0, w, e)):
        n = k * 7 % (most + 1)
        img[y + g.integers(0, min(e, h - y), n), x + g.integers(0, min(e, w - x), n)] += g.uniform(150, 900, n)
        if k % 3 == 0:
            yy, xx = np.mgrid[y:min(y + e, h), x:min(x + e, w)]
            s = 1.2 + 0.25 * (k % 17)
            img[yy, xx] += 40000.0 * np.exp(-((yy - y - e / 2) ** 2 + (xx - x - e / 2) ** 2) / (2 * s * s))
    _check(img.astype(F32), niter=4, sepmed=sepmed)
