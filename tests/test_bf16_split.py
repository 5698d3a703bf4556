"""The three-part bf16 split of the FP32 M2L, emulated: exact for every FP32
number after the scaling that the kernels apply (2^24 below 2^100, 2^-4 from
there on), and not without it.
"""
import numpy as np


def _bf16(x):
    """Round float32 to bf16, ties to even, kept as float32; subnormals kept."""
    u = x.view(np.uint32).astype(np.uint64)
    return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(np.float32)


def _parts(x):
    p = []
    with np.errstate(invalid="ignore"):
        for _ in range(3):
            h = _bf16(x)
            x = (x - h).astype(np.float32)
            p.append(h.astype(np.float64))
    return p


def _numbers():
    rng = np.random.default_rng(5)
    m = rng.integers(0, 1 << 23, 4000, dtype=np.uint32)
    m[:3] = [0, 1, (1 << 23) - 1]
    bits = (np.arange(0, 255, dtype=np.uint32)[:, None] << 23) | m  # every exponent, subnormals among them
    return bits.ravel().view(np.float32)


def test_scaled_split_is_exact():
    x = _numbers()
    s = np.where(np.abs(x) < 2.0**100, np.float32(2.0**24), np.float32(2.0**-4)).astype(np.float32)
    y = x * s
    assert np.isfinite(y).all() and np.array_equal(y.astype(np.float64), x.astype(np.float64) * s)
    assert np.array_equal(sum(_parts(y)), y.astype(np.float64))


def test_unscaled_split_is_not():
    x = _numbers()
    with np.errstate(invalid="ignore"):
        bad = ~(sum(_parts(x)) == x.astype(np.float64))
    # lost: the last bits below 2^-109, and overflow at the top of the range
    assert bad[np.abs(x) < 2.0**-110].any() and bad[np.abs(x) > 3.39e38].any()
    assert not bad[(np.abs(x) >= 2.0**-109) & (np.abs(x) < 3.38e38)].any()
