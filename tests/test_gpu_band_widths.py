"""Band SpMV with half-widths that no instance is unrolled for: every remainder of the eight diagonals read at a time, matrices narrower than the
band, edge rows; NaN in every padding slot, which must not reach a result; small integers bit for bit."""
import numpy as np
import pytest

from paper_2407_13726_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("w", [0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 31, 32, 40])
def test_widths(gpu, oracle, w, f64):
    t = np.float64 if f64 else np.float32
    for n in sorted({1, 2, max(1, w), w + 1, 2 * w + 1, 2 * w + 3, 255, 257, 1000}):
        D = inputs.small_int(9000 + n + w, -3, 3, 2 * w + 1, n).astype(t)
        for d in range(-w, w + 1):
            D[d + w, [i for i in range(n) if not 0 <= i + d < n]] = np.nan
        x = inputs.small_int(9100 + n + w, -3, 3, n).astype(t)
        want, _ = (oracle.band_spmv_f64 if f64 else oracle.band_spmv)(n, w, D.ravel(), x)
        y = gpu.up(np.full(n, np.nan, dtype=t))
        (gpu.d.band_spmv_f64 if f64 else gpu.d.band_spmv_f32)(n, w, gpu.up(D.ravel()), gpu.up(x), y)
        assert gpu.down(y).tobytes() == want.astype(t).tobytes(), n
