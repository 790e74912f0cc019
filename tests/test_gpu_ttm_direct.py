"""TTM_UT for few packed rows: edges of its windows of 16 values of l, of its tiles (32 or 16 rows, 32 columns) and of the choices of two or four wavefronts
and of the kernels for more rows; small integers bit for bit, row strides of C, values that are not finite."""
import numpy as np
import pytest

from paper_2407_13726_amd import inputs

pytestmark = pytest.mark.gpu


def operands(n, Q, K, ldc, f64):
    t = np.float64 if f64 else np.float32
    return (inputs.small_int(8000 + n + Q, -3, 3, n * (n + 1) // 2 * Q).astype(t), inputs.small_int(8100 + K + Q, -3, 3, K, ldc).astype(t))


def ttm(gpu, n, Q, K, ldc, B, C):
    A = gpu.up(np.full(n * (n + 1) // 2 * K, np.nan, dtype=B.dtype))
    (gpu.d.ttm_ut_f64 if B.dtype == np.float64 else gpu.d.ttm_ut_f32)(n, Q, K, gpu.up(B), gpu.up(C), ldc, A)
    return gpu.down(A)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,Q,K,ldc", [(1, 16, 1, 16), (1, 15, 1, 15), (2, 17, 3, 20), (5, 31, 33, 31), (7, 32, 32, 32), (8, 48, 31, 48), (8, 49, 65, 49), (24, 500, 100, 501),
                                       (30, 47, 64, 47), (33, 261, 112, 261), (63, 100, 20, 100), (100, 33, 40, 33), (130, 65, 100, 65), (150, 40, 120, 40),
                                       (202, 20, 64, 20), (203, 20, 64, 20), (180, 50, 62, 50), (256, 16, 30, 16), (260, 35, 48, 35),
                                       (260, 18, 49, 18)])
def test_exact_on_integers(gpu, oracle, n, Q, K, ldc, f64):
    B, C = operands(n, Q, K, ldc, f64)
    want, _ = (oracle.ttm_ut_f64 if f64 else oracle.ttm_ut)(n, Q, K, B, np.ascontiguousarray(C[:, :Q]))
    assert ttm(gpu, n, Q, K, ldc, B, C).tobytes() == want.astype(B.dtype).tobytes()


@pytest.mark.parametrize("f64,n,Q,K", [(True, 142, 32, 33), (True, 143, 32, 33), (True, 201, 128, 64), (True, 202, 128, 64), (True, 160, 144, 100), (True, 161, 144, 100),
                                       (True, 308, 65, 48), (True, 308, 63, 48), (True, 312, 256, 34), (True, 312, 257, 34), (True, 220, 48, 32), (False, 201, 200, 64),
                                       (False, 202, 200, 64)])
def test_both_sides_of_the_choice(gpu, oracle, f64, n, Q, K):
    """By remainder of Q, number of tiles and columns."""
    test_exact_on_integers(gpu, oracle, n, Q, K, Q, f64)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("Q", [16, 37, 260])
@pytest.mark.parametrize("value", [np.nan, np.inf, 3e38])
def test_values_that_are_not_finite_stay_where_they_belong(gpu, Q, f64, value):
    n, K = 12, 40
    B, C = operands(n, Q, K, Q, f64)
    B, C = np.abs(B) + 1, np.abs(C) + 1
    whole = ttm(gpu, n, Q, K, Q, B, C).reshape(-1, K)
    for l in (0, Q - 17 if Q > 16 else 3, Q - 1):
        bad = B.copy().reshape(-1, Q)
        bad[33, l] = value
        got = ttm(gpu, n, Q, K, Q, bad.ravel(), C).reshape(-1, K)
        assert np.array_equal(np.delete(got, 33, 0), np.delete(whole, 33, 0))
        with np.errstate(all="ignore"):
            want = (bad[33].astype(np.float64) @ C.astype(np.float64).T).astype(B.dtype)
        assert np.array_equal(np.isnan(got[33]), np.isnan(want)) and np.allclose(got[33], want, rtol=1e-6, equal_nan=True)
        bad = C.copy()
        bad[35, l] = value
        got = ttm(gpu, n, Q, K, Q, B, bad).reshape(-1, K)
        assert np.array_equal(np.delete(got, 35, 1), np.delete(whole, 35, 1))
        with np.errstate(all="ignore"):
            want = (B.reshape(-1, Q).astype(np.float64) @ bad[35].astype(np.float64)).astype(B.dtype)
        assert np.array_equal(np.isnan(got[:, 35]), np.isnan(want)) and np.allclose(got[:, 35], want, rtol=1e-6, equal_nan=True)


@pytest.mark.parametrize("n,Q,K", [(10, 16, 5), (30, 20, 40), (60, 25, 100), (60, 32, 500), (80, 31, 256)])
def test_few_terms_have_the_products_of_the_type(gpu, n, Q, K):
    """Where a row of C has one element, a result is one rounded product in single precision, with every bit."""
    B, C = inputs.uniform(8200 + n, n * (n + 1) // 2 * Q), np.zeros((K, Q), dtype=np.float32)
    l = np.arange(K) % Q
    C[np.arange(K), l] = inputs.uniform(8300 + n, K)
    got = ttm(gpu, n, Q, K, Q, B, C).reshape(-1, K)
    assert np.array_equal(got, B.reshape(-1, Q)[:, l] * C[np.arange(K), l])
