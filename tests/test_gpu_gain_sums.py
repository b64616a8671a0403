"""GPU tests of the gain estimate's sums and medians where its register
windows and its near histogram end: values across many powers of two and both
signs (most of them outside the window), frames whose pixel count is not a
multiple of four, fewer pixels than a wave, medians that move further between
rounds than the near histogram reaches, and integer values with ties.  The
per-iteration gains must equal the oracle's binary32 gains exactly."""

import numpy as np
import pytest

from gpu_common import assert_bits_equal, host_threads, lac, to_dev

pytestmark = pytest.mark.gpu

F32 = np.float32


def _values(case, h, w):
    g = np.random.Generator(np.random.PCG64(len(case) + h))
    if case == "octaves":  # 2^-20 .. 2^20, both signs
        return (g.choice([-1.0, 1.0], (h, w)) * np.exp2(g.uniform(-20, 20, (h, w)))).astype(F32)
    if case == "centred":  # noise about zero: the keys around the median are dense
        return g.normal(0.01, 12.0, (h, w)).astype(F32)
    if case == "skewed":  # clipping moves the median far in every round
        return (50.0 + g.exponential(30.0, (h, w)) ** 2).astype(F32)
    if case == "integer":
        return g.poisson(90.0, (h, w)).astype(F32)
    img = g.normal(300.0, 9.0, (h, w))  # "tiny"/"plain" values with a few zeros and denormals
    img.reshape(-1)[::7] = 0.0
    img.reshape(-1)[::11] = 1e-41
    return img.astype(F32)


@pytest.mark.parametrize("shape", [(3, 5), (65, 67), (257, 255), (1027, 1031)])
@pytest.mark.parametrize("case", ["octaves", "centred", "skewed", "integer", "zeros"])
def test_gains_equal_the_oracle(case, shape):
    import oracle
    L = lac()
    img = _values(case, *shape)
    r = oracle.lacosmic(img, 0.0, 4.0, 4.5, 0.3, 5.0, 2, nthreads=host_threads(), estimate_gain=True)
    m, c, st = L.run_ex(to_dev(img), L.make_params(0.0, 4.0, niter=2, estimate_gain=True))
    assert [F32(st.gain[k]) for k in range(2)] == [F32(x) for x in r["gains"]]
    assert_bits_equal(m.cpu().numpy(), r["mask"], "mask")
    assert_bits_equal(c.cpu().numpy(), r["clean"], "clean")
