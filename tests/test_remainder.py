"""remainder_of (wave_common.hpp), the draw's hash mod legal_count in floats, restated in numpy: right for every count the games can have,
also with reciprocals one unit in the last place off either way, as the hardware's instruction may give them."""
import numpy as np
import pytest


def remainder_of(n, d, ulp):
    f32 = np.float32
    f = (f32(1) / d.astype(f32)).view(np.int32) + np.int32(ulp)
    f = f.view(f32)
    q = np.minimum(n.astype(f32) * f, f32(4294967040.0)).astype(np.uint64).astype(np.uint32)
    left = (n - q * d).view(np.int32)
    # the fused multiply-add rounds once: exact in 64 bits, then rounded
    v = (left.astype(f32).astype(np.float64) * f.astype(np.float64) + (f32(0.5) * f).astype(np.float64)).astype(f32)
    return (left - np.floor(v).astype(np.int32) * d.astype(np.int32)).view(np.uint32)


@pytest.mark.parametrize("ulp", [-1, 0, 1])
def test_every_count(ulp):
    rng = np.random.default_rng(5)
    for count in list(range(1, 1025)):
        n = rng.integers(0, 1 << 32, 500, dtype=np.uint32)
        multiple = n // np.uint32(count) * np.uint32(count)
        edge = np.arange(500, dtype=np.uint32)
        n = np.concatenate([n, multiple, multiple - np.uint32(1), multiple + np.uint32(count - 1), edge, ~edge])
        assert np.array_equal(remainder_of(n, np.full_like(n, count), ulp), n % np.uint32(count)), count
