"""The FP32 filters in front of the exact acceptance predicate: what they call certain is
certain.  The logarithm that they use is compared with FP64 at every float that can occur,
and the bounds with 64-bit-mantissa logarithms over all magnitudes of a draw."""
import numpy as np
import pytest

from test_gpu_parity import rw  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def bits(x):
    return int(np.float32(x).view(np.uint32))


def test_log2_within_its_bound_at_every_float(rw):
    # 2^-60 <= u <= 1, by binary exponent (a draw with w > 0 has u >= 2^-32)
    worst = [rw.rewl_probe_log2(bits(2.0 ** -e), 1 << 23) for e in range(60, 0, -1)] + [rw.rewl_probe_log2(bits(1.0), 1)]
    assert max(worst) <= 1.0 and worst[-1] == 0.0
    # the comparison is one: the FP64 logarithm it takes is that of the host at the ends
    assert 0.5 < max(worst)
    for e in (1, 17, 32):
        assert rw.rewl_probe_log2(bits(2.0 ** -e), 1) == 0.0


@pytest.mark.parametrize("band", [2.0 ** -40, 2.0 ** -13, 2.0 ** -2])
def test_bounds_are_certain(rw, band):
    rng = np.random.default_rng(7)
    n = 1 << 20
    # words of every magnitude, their neighbours, and draws as they come
    small = [max(0, min(2 ** 32 - 1, (1 << e) + d)) for e in range(33) for d in range(-3, 4)]
    w = np.concatenate([np.repeat(small, 64), rng.integers(0, 1 << 32, n), (2.0 ** rng.uniform(0, 32, n)).astype(np.int64)])
    z = rng.integers(0, 1 << 32, len(w))
    z[:: 5] = 0
    z[1:: 5] = 2 ** 32 - 1
    z[2:: 5] = rng.integers(0, 1 << 14, len(z[2:: 5]))
    zw = np.stack([z, np.minimum(w, 2 ** 32 - 1)], axis=1).astype(np.uint32)
    lo, hi, up, low = (v.astype(np.longdouble) for v in rw.rewl_probe_bounds(zw, band).T)
    u53 = ((zw[:, 1].astype(np.uint64) << np.uint64(32)) | zw[:, 0]) >> np.uint64(11)
    some = u53 > 0
    with np.errstate(divide="ignore"):
        lg = np.log(u53.astype(np.longdouble)) - 53 * np.log(np.longdouble(2))
    # wave: delta > hi accepts, delta < lo rejects by the FP64 test with this band
    assert (hi[some] > lg[some] + band).all() and (lo[some] < lg[some] - band).all()
    # lane: the same for a delta rounded to FP32 (2^-19 up to 64)
    assert (up[some] > lg[some] + band + 2.0 ** -19).all() and (low[some] < lg[some] - band - 2.0 ** -19).all()
    # a draw of 0 accepts every finite delta and no infinite one
    tiny = -np.finfo(np.float32).max
    assert (~some).any() and (hi[~some] == np.inf).all() and (lo[~some] == tiny).all()
    assert (up[~some] == tiny).all() and (low[~some] <= tiny).all()
