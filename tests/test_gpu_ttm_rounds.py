"""TTM_UT in rounds of tiles: the larger tiles, rows that end inside a tile, rows left to a launch of their own, whole and ragged columns and steps, and sub-tiles that are not
finite in each of them."""
import numpy as np
import pytest

from paper_2407_13726_amd import inputs

pytestmark = pytest.mark.gpu


def ttm(gpu, n, Q, K, B, C):
    A = gpu.up(np.full(n * (n + 1) // 2 * K, np.nan, dtype=np.float32))
    gpu.d.ttm_ut_f32(n, Q, K, gpu.up(B), gpu.up(C), Q, A)
    return gpu.down(A).reshape(-1, K)


# n: 256 has 32896 rows, 257 tiles of 128 (one more than a round or two); 220 and 300 end inside a tile; 361 to 363 with one column block are a round of 256 x 128, or two of
# 128 x 128, and a few rows.  Tiles of 128 rows in one launch: 256 with Q <= 64, 257, 363 with Q = 36, 400; with the rest apart: 256 with Q = 100; of 256 rows: 220, 300, 361, 512 (few
# steps and much output); with the rest apart: 256 with Q = 120, 362, 363 with Q = 128
@pytest.mark.parametrize("n,Q,K", [(220, 300, 200), (256, 16, 128), (256, 33, 129), (256, 100, 65), (256, 64, 256), (257, 20, 97), (300, 100, 128), (300, 35, 72),
                                   (361, 40, 128), (363, 36, 100), (400, 48, 96), (256, 120, 256), (362, 70, 100), (363, 128, 256), (512, 10, 500)])
def test_exact_on_integers(gpu, n, Q, K):
    rows = n * (n + 1) // 2
    B, C = inputs.small_int(8400 + n, -3, 3, rows * Q).astype(np.float32), inputs.small_int(8500 + K, -3, 3, K, Q).astype(np.float32)
    got = ttm(gpu, n, Q, K, B, C)
    want = (gpu.up(B).view(rows, Q).double() @ gpu.up(C).double().t().contiguous()).float().cpu().numpy()
    assert got.tobytes() == want.tobytes() or np.array_equal(got, want)


@pytest.mark.parametrize("n,Q,K", [(220, 300, 200), (256, 64, 256), (256, 100, 100), (362, 70, 100)])
@pytest.mark.parametrize("value", [np.nan, np.inf, 3e38])
def test_values_that_are_not_finite_stay_where_they_belong(gpu, n, Q, K, value):
    rows = n * (n + 1) // 2
    B, C = inputs.small_int(8600 + n, 1, 3, rows, Q).astype(np.float32), inputs.small_int(8700 + K, 1, 3, K, Q).astype(np.float32)
    whole = ttm(gpu, n, Q, K, B.ravel(), C)
    at = [0, 300, rows // 2, rows - 1]
    bad = B.copy()
    bad[at, Q // 2] = value
    got = ttm(gpu, n, Q, K, bad.ravel(), C)
    assert np.array_equal(np.delete(got, at, 0), np.delete(whole, at, 0))
    with np.errstate(all="ignore"):
        want = (bad[at].astype(np.float64) @ C.astype(np.float64).T).astype(np.float32)
    assert np.array_equal(np.isnan(got[at]), np.isnan(want)) and np.allclose(got[at], want, rtol=1e-6, equal_nan=True)
