"""Triangular products in one launch: edges of its row blocks (32, 16), windows (16), column blocks (32) and of the choice between 4, 8 and 16
wavefronts and the tiles of the large products; small integers bit for bit, row strides, equal bits on equal calls, values that are not finite."""
import numpy as np
import pytest

from paper_2407_13726_amd import inputs

pytestmark = pytest.mark.gpu


def operands(n, m, ld, f64, lo, hi):
    t = np.float64 if f64 else np.float32
    return inputs.small_int(6000 + n + m, lo, hi, n * (n + 1) // 2).astype(t), inputs.small_int(6100 + n + m, lo, hi, n, ld).astype(t)


def product(gpu, n, m, ld, U, B):
    C = gpu.up(np.full((n, ld), np.nan, dtype=U.dtype))
    getattr(gpu.d, "trmm_f64" if U.dtype == np.float64 else "trmm_f32")(n, m, gpu.up(U), gpu.up(B), ld, C, ld)
    return gpu.down(C)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,m,ld", [(63, 5, 5), (64, 1, 3), (64, 33, 33), (65, 32, 32), (79, 31, 40), (80, 64, 64), (97, 2, 2), (255, 65, 65), (257, 100, 101),
                                    (499, 130, 130), (500, 33, 33), (1000, 225, 225), (1000, 7, 7), (1001, 130, 130), (1100, 16, 16), (1101, 16, 16), (1536, 8, 8),
                                    (1537, 8, 8), (1999, 40, 40), (2001, 20, 20), (2048, 32, 32), (2049, 32, 32), (100, 2048, 2048), (100, 2049, 2049), (3500, 40, 40),
                                    (3501, 40, 40)])
def test_exact_on_integers(gpu, oracle, n, m, ld, f64):
    U, B = operands(n, m, ld, f64, -3, 3)
    want, _ = (oracle.trmm_f64 if f64 else oracle.trmm)(n, m, U, np.ascontiguousarray(B[:, :m]))
    got = product(gpu, n, m, ld, U, B)
    assert got[:, :m].tobytes() == want.astype(U.dtype).tobytes()
    assert np.isnan(got[:, m:]).all()


@pytest.mark.parametrize("n,m", [(256, 100), (1500, 100), (3000, 40)])
def test_equal_calls_give_equal_bits(gpu, n, m):
    for U, B in ((inputs.uniform(6200, n * (n + 1) // 2), inputs.uniform(6201, n, m)), (inputs.uniform64(6202, n * (n + 1) // 2), inputs.uniform64(6203, n * m).reshape(n, m))):
        got = [product(gpu, n, m, m, U, B).tobytes() for _ in range(3)]
        assert got[0] == got[1] == got[2]


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,m", [(70, 5), (100, 40), (1001, 33)])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_values_that_are_not_finite_stay_where_they_belong(gpu, n, m, value, f64):
    """A row of B reaches the rows of C up to its own, an element of U one row of C; every other element is as without it."""
    U, B = operands(n, m, m, f64, 1, 3)
    whole = product(gpu, n, m, m, U, B)
    for k in (0, 5, 17, n // 2, n - 3, n - 1):
        bad = B.copy()
        bad[k, m // 2] = value
        got = product(gpu, n, m, m, U, bad)
        touched = np.zeros((n, m), dtype=bool)
        touched[:k + 1, m // 2] = True
        assert np.array_equal(got[~touched], whole[~touched]), k
        assert (np.isnan(got[touched]) if np.isnan(value) else np.isposinf(got[touched])).all(), k
    i = n // 3
    bad = U.copy()
    bad[i * n - i * (i - 1) // 2 + 2] = value  # U(i, i + 2)
    got = product(gpu, n, m, m, bad, B)
    assert np.array_equal(np.delete(got, i, 0), np.delete(whole, i, 0))
    assert (np.isnan(got[i]) if np.isnan(value) else np.isposinf(got[i])).all()


@pytest.mark.parametrize("scale", [2.0 ** 60, 2.0 ** -100, 3e38])
def test_values_beyond_the_split(gpu, oracle, scale):
    n, m = 130, 40
    U, B = operands(n, m, m, False, 1, 3)
    U = (U * np.float32(scale / 3)).astype(np.float32)
    with np.errstate(all="ignore"):
        want, _ = oracle.trmm(n, m, U, B)
    got, want = product(gpu, n, m, m, U, B), want.astype(np.float32)
    assert np.array_equal(np.isinf(got), np.isinf(want))
    ok = np.isfinite(want)
    assert np.allclose(got[ok], want[ok], rtol=1e-6, atol=0)


@pytest.mark.parametrize("n,m", [(64, 2), (65, 32), (130, 17), (1000, 8), (1536, 32), (2048, 9), (3000, 5)])
def test_few_columns_have_the_products_of_the_type(gpu, n, m):
    """A row of C that meets one row of B is one rounded product in single precision, with every bit."""
    U, B = inputs.uniform(6300 + n, n * (n + 1) // 2), np.zeros((n, m), dtype=np.float32)
    k = n - 1 - np.arange(m) % 3 * (n // 3)  # the one row that column c meets
    B[k, np.arange(m)] = inputs.uniform(6400 + n, m)
    got = product(gpu, n, m, m, U, B)
    i = np.arange(n)
    for c in range(m):
        rows = i[i <= k[c]]
        assert np.array_equal(got[rows, c], U[rows * n - rows * (rows - 1) // 2 + k[c] - rows] * B[k[c], c])
        assert not got[k[c] + 1:, c].any()


@pytest.mark.parametrize("f64,n,m", [(False, 64, 2048), (False, 976, 2048), (False, 3500, 163), (False, 3500, 8), (True, 64, 2048), (True, 644, 2048), (True, 3500, 69), (True, 2000, 32),
                                     (True, 1100, 16)])
def test_one_writer_up_to_the_edges_of_the_choice(gpu, f64, n, m):
    uniform = inputs.uniform64 if f64 else inputs.uniform
    U, B = uniform(6500 + n, n * (n + 1) // 2), uniform(6600 + n, n * m).reshape(n, m)
    got = [product(gpu, n, m, m, U, B).tobytes() for _ in range(3)]
    assert got[0] == got[1] == got[2]


@pytest.mark.parametrize("n", [199, 200, 201, 1200, 1201])
@pytest.mark.parametrize("m", [1, 31, 32])
def test_wavefronts_by_rows(gpu, oracle, n, m):
    """Up to 32 columns in single precision: four, eight or sixteen wavefronts."""
    test_exact_on_integers(gpu, oracle, n, m, m, False)
