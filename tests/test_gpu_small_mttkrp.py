"""MTTKRP of small tensors: sizes around its groups of eight k, its tiles of 64 columns and the sizes where the blocks take over; small
integers bit for bit, row strides, equal bits on equal calls, and factor rows above a slice that must not reach it."""
import numpy as np
import pytest

from paper_2407_13726_amd import inputs

pytestmark = pytest.mark.gpu


def tet(n):
    return n * (n + 1) * (n + 2) // 6


def mttkrp(gpu, n, R, ld, A, B, C):
    M = gpu.up(np.full((n, ld), np.nan, dtype=A.dtype))
    (gpu.d.tet_mttkrp_f64 if A.dtype == np.float64 else gpu.d.tet_mttkrp_f32)(n, R, gpu.up(A), gpu.up(B), ld, gpu.up(C), ld, M, ld)
    return gpu.down(M)


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,R,ld", [(1, 1, 1), (2, 3, 3), (3, 65, 65), (7, 5, 6), (8, 64, 64), (9, 2, 2), (15, 33, 33), (16, 128, 128), (17, 1, 4), (48, 20, 20), (72, 7, 7),
                                    (73, 40, 40), (80, 32, 32), (81, 9, 9), (87, 8, 8), (88, 32, 32), (89, 32, 32), (104, 33, 33), (110, 90, 91), (111, 70, 70)])
def test_exact_on_integers(gpu, oracle, n, R, ld, f64):
    t = np.float64 if f64 else np.float32
    A = inputs.small_int(7000 + n, -2, 2, tet(n)).astype(t)
    B, C = (inputs.small_int(7100 + n + s, -2, 2, n, ld).astype(t) for s in (0, 1))
    want, _ = (oracle.tet_mttkrp_f64 if f64 else oracle.tet_mttkrp)(n, R, A, np.ascontiguousarray(B[:, :R]), np.ascontiguousarray(C[:, :R]))
    got = mttkrp(gpu, n, R, ld, A, B, C)
    assert got[:, :R].tobytes() == want.astype(t).tobytes()
    assert np.isnan(got[:, R:]).all()


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,R", [(64, 513), (65, 512), (65, 513), (80, 512), (80, 513), (88, 600), (100, 512), (100, 513), (101, 192), (101, 193)])
def test_many_columns(gpu, oracle, n, R, f64):
    """Both sides of the lines that columns draw between the kernels."""
    test_exact_on_integers(gpu, oracle, n, R, R, f64)


@pytest.mark.parametrize("n,R", [(50, 20), (100, 64)])
def test_equal_calls_give_equal_bits(gpu, n, R):
    A, B, C = inputs.normal(7200, tet(n)), inputs.normal(7201, n, R), inputs.normal(7202, n, R)
    assert len({mttkrp(gpu, n, R, R, A, B, C).tobytes() for _ in range(3)}) == 1


@pytest.mark.parametrize("n", [9, 40, 88])
def test_factor_rows_of_smaller_index_do_not_reach_a_slice(gpu, n):
    A, B, C = (np.abs(inputs.small_int(7300 + s, 1, 3, *shape)).astype(np.float32) for s, shape in enumerate(((tet(n),), (n, 5), (n, 5))))
    whole = mttkrp(gpu, n, 5, 5, A, B, C)
    for at in (0, n // 2, n - 2):
        for bad, other in ((B, C), (C, B)):
            spoilt = bad.copy()
            spoilt[at] = np.nan
            got = mttkrp(gpu, n, 5, 5, A, spoilt, other) if bad is B else mttkrp(gpu, n, 5, 5, A, other, spoilt)
            assert np.array_equal(got[at + 1:], whole[at + 1:]) and np.isnan(got[:at + 1]).all()


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n,R", [(2, 3), (9, 5), (40, 33), (88, 20), (130, 20)])
def test_a_meets_b_before_c(gpu, n, R, f64):
    """(A(i,j,k) B(j,r)) C(k,r), as the rule has it: what cancels in magnitude between A and B neither overflows nor vanishes, on both sides of
    the line between the kernels."""
    t, e = (np.float64, 160) if f64 else (np.float32, 20)
    for a, b, c in ((10.0 ** e, 10.0 ** -e, 10.0 ** e), (10.0 ** -e, 10.0 ** e, 10.0 ** -e)):
        A, B, C = np.full(tet(n), a, dtype=t), np.full((n, R), b, dtype=t), np.full((n, R), c, dtype=t)
        got = mttkrp(gpu, n, R, R, A, B, C)
        terms = np.array([(n - i) * (n - i + 1) // 2 for i in range(n)], dtype=np.float64)
        assert np.allclose(got, (terms * c)[:, None], rtol=tet(n) * np.finfo(t).eps, atol=0)
