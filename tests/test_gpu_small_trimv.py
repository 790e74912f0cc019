"""Products of one small packed triangle by the kernel that writes every output once: sizes around its blocks of 8 and 16 outputs, a last block that is moved
back, and the sizes where the panels take over; small integers bit for bit, and the same bits on every call."""
import numpy as np
import pytest

from paper_2407_13726_amd import inputs

pytestmark = pytest.mark.gpu

FORMS = [("symv", False, 2), ("symv_lower", True, 2), ("trmv_t", False, 1), ("trmv_lower", True, 0), ("trmv_lower_t", True, 1)]
SIZES = [1, 2, 7, 8, 9, 15, 16, 17, 63, 65, 255, 257, 511, 700, 1023, 2047, 2048, 2049, 2063, 2065, 3071, 3073, 4095, 4096, 4097]


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n", SIZES)
def test_small_triangles(gpu, oracle, n, f64):
    t = np.float64 if f64 else np.float32
    T = inputs.small_int(5000 + n, -3, 3, n * (n + 1) // 2).astype(t)
    x = inputs.small_int(5100 + n, -3, 3, n).astype(t)
    dT, dx = gpu.up(T), gpu.up(x)
    for name, lower, mode in FORMS:
        want, _ = (oracle.trimv_f64 if f64 else oracle.trimv)(n, T, x, lower=lower, mode=mode)
        y = gpu.up(np.full(n, np.nan, dtype=t))
        getattr(gpu.d, name + ("_f64" if f64 else "_f32"))(n, dT, dx, y)
        assert gpu.down(y).tobytes() == want.astype(t).tobytes(), name


@pytest.mark.parametrize("n", [300, 1999, 3333])
def test_equal_calls_give_equal_bits(gpu, n):
    T, x = gpu.up(inputs.normal(5200 + n, n * (n + 1) // 2)), gpu.up(inputs.normal(5300 + n, n))
    got = []
    for _ in range(3):
        y = gpu.up(np.full(n, np.nan, dtype=np.float32))
        gpu.d.symv_f32(n, T, x, y)
        got.append(gpu.down(y).tobytes())
    assert got[0] == got[1] == got[2]


@pytest.mark.parametrize("n", [40, 2500])
def test_elements_outside_the_triangle_meet_no_vector_element(gpu, oracle, n):
    """An infinite element of x reaches every output of the full symmetric product, but only its own half of the triangular ones."""
    T = np.abs(inputs.small_int(5400 + n, 1, 3, n * (n + 1) // 2)).astype(np.float32)
    x = inputs.small_int(5500 + n, 1, 3, n).astype(np.float32)
    x[n // 3] = np.inf
    for (name, lower, mode), keep in zip(FORMS[2:], (slice(0, n // 3), slice(0, n // 3), slice(n // 3 + 1, n))):
        want, _ = oracle.trimv(n, T, x, lower=lower, mode=mode)
        y = gpu.up(np.full(n, np.nan, dtype=np.float32))
        getattr(gpu.d, name + "_f32")(n, gpu.up(T), gpu.up(x), y)
        got = gpu.down(y)
        assert np.array_equal(got[keep], want[keep]) and np.isfinite(got[keep]).all(), name
        assert np.isinf(np.delete(got, np.r_[keep])).all(), name
