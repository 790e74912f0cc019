"""Third-order polynomial-regression tensor: every kernel and both ways of dealing out the samples, at the edges of steps (16, 32 samples),
tiles (8 or 16 rows, 32 columns, 4 or 16 slices) and row strides; small integers bit for bit, which is exact in any order."""
import numpy as np
import pytest

from paper_2407_13726_amd import inputs

pytestmark = pytest.mark.gpu


def tet(n):
    return n * (n + 1) * (n + 2) // 6


FEW = [(1, 1, 1), (2, 7, 7), (15, 33, 40), (15, 70, 70)]                       # fewer than a step of samples
DIRECT = [(16, 1, 1), (16, 9, 9), (17, 2, 5), (31, 31, 31), (33, 8, 8), (47, 32, 33), (129, 16, 16), (257, 63, 64), (700, 25, 25),
          (300, 97, 97), (1000, 65, 65), (5001, 17, 17), (16, 129, 129), (40, 200, 201)]  # one share and several
TWO_TILES = [(200, 152, 152), (767, 129, 130), (799, 130, 130)]                # single precision: two tiles, two and four wavefronts
STAGED = [(4500, 105, 107), (4836, 112, 112)]                                  # single precision: shared columns


@pytest.mark.parametrize("N,d,ld", FEW + DIRECT + TWO_TILES + STAGED)
def test_pr_a3_f32(gpu, oracle, N, d, ld):
    B = inputs.small_int(2500 + N + d, -2, 2, N, ld)
    want, _ = oracle.pr_a3(np.ascontiguousarray(B[:, :d]))
    out = gpu.empty(tet(d))
    gpu.d.pr_a3_f32(N, d, gpu.up(B), ld, out)
    assert gpu.down(out).tobytes() == want.tobytes()
    if N * tet(d) < 3 * 10 ** 8:
        B = inputs.normal(2600 + N + d, N, ld)
        want, scale = oracle.pr_a3(np.ascontiguousarray(B[:, :d]))
        gpu.d.pr_a3_f32(N, d, gpu.up(B), ld, out)
        # two rounded products (2^-23; the split leaves out 2^-23 more) and at most one rounding by 2^-24 of the sum of the |products| per
        # sample; the split's accumulator cuts off up to 2^-23 once in 16 samples for each of its six products, which is less
        err = np.abs(gpu.down(out).astype(np.float64).ravel() - want.ravel())
        assert (err <= (N + 4) * 2.0 ** -24 * scale.ravel()).all()


@pytest.mark.parametrize("N,d,ld", FEW + DIRECT + TWO_TILES)
def test_pr_a3_f64(gpu, oracle, N, d, ld):
    B = inputs.small_int(2700 + N + d, -2, 2, N, ld).astype(np.float64)
    want, _ = oracle.pr_a3_f64(np.ascontiguousarray(B[:, :d]))
    out = gpu.up(np.full(tet(d), np.nan))
    gpu.d.pr_a3_f64(N, d, gpu.up(B), ld, out)
    assert gpu.down(out).tobytes() == want.tobytes()


@pytest.mark.parametrize("N,d", [(15, 20), (60, 40), (4500, 105)])
@pytest.mark.parametrize("value", [np.nan, np.inf, 3e38])
def test_one_sample_that_is_not_finite(gpu, oracle, N, d, value):
    """Only the elements that meet the value are touched, in the one way that IEEE arithmetic has it; every other is as without it."""
    B = inputs.small_int(2800 + N, 1, 2, N, d)
    B[N - 1, d // 2] = value
    with np.errstate(all="ignore"):
        want, _ = oracle.pr_a3(B)
    out = gpu.empty(tet(d))
    gpu.d.pr_a3_f32(N, d, gpu.up(B), d, out)
    got, want = gpu.down(out).ravel(), want.ravel()
    meets = np.array([d // 2 in (i, j, k) for i in range(d) for j in range(i, d) for k in range(j, d)])
    assert np.array_equal(got[~meets], want[~meets])
    if np.isnan(value):
        assert np.isnan(got[meets]).all()
    elif np.isinf(value):
        assert np.isinf(got[meets]).all() and (got[meets] > 0).all()
    else:  # value, 2 value and 4 value: the last two are beyond the range
        ok = np.isfinite(want[meets].astype(np.float32))
        assert np.allclose(got[meets][ok], want[meets][ok], rtol=1e-6)
