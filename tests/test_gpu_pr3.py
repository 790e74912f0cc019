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


ORDER = [(1, 5, 5), (3, 20, 20), (15, 33, 40), (16, 33, 33), (40, 70, 71), (300, 97, 97), (4500, 105, 107)]


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("N,d,ld", ORDER)
def test_products_are_formed_in_the_order_of_the_rule(gpu, N, d, ld, f64):
    """(B(x,i) B(x,j)) B(x,k): a pair that cancels in magnitude comes first where i and j have it, so that the third factor neither overflows nor
    vanishes; pairs that overflow by themselves give infinity.  (Pairs below the normal range may come out closer than the type has them.)"""
    t, big, small, nothing = (np.float64, 515, -510, -540) if f64 else (np.float32, 66, -62, -76)
    at = [d // 4, d // 2, d - 1]
    for values in ((big, small, big), (nothing, big, nothing)):
        B = np.zeros((N, ld), dtype=t)
        B[N // 2, :d] = 1.5
        B[N // 2, at] = np.ldexp(1.0, values)
        b = B[N // 2, :d]
        with np.errstate(all="ignore"):
            pair = (b[:, None] * b[None, :])[:, :, None]
            cube = pair * b
        k = np.arange(d)
        wanted = (k[:, None] <= k[None, :])[:, :, None] & (k[None, :, None] <= k[None, None, :])
        want, pair = cube[wanted], np.broadcast_to(pair, cube.shape)[wanted]
        out = gpu.up(np.full(tet(d), np.nan, dtype=t))
        (gpu.d.pr_a3_f64 if f64 else gpu.d.pr_a3_f32)(N, d, gpu.up(B), ld, out)
        got, tiny = gpu.down(out), np.finfo(t).tiny
        assert np.array_equal(np.isposinf(got), np.isposinf(want)) and not np.isnan(got).any()
        normal = np.isfinite(want) & (pair >= tiny)
        # one term of two rounded products (the split leaves out up to 2^-22 of it); below the normal range products lose bits or vanish
        assert np.allclose(got[normal], want[normal], rtol=2.0 ** -20, atol=tiny)


def expected(b):
    """(b_i b_j) b_k of one row of samples, packed: the pair rounded to its type, the product with b_k in double precision; and where they stand."""
    k = np.arange(len(b))
    wanted = (k[:, None] <= k[None, :])[:, :, None] & (k[None, :, None] <= k[None, None, :])
    return ((b[:, None] * b[None, :]).astype(np.float64)[:, :, None] * b.astype(np.float64))[wanted]


@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("N", [1, 4, 5, 8, 9, 15])
def test_strips_of_few_samples(gpu, oracle, N, f64):
    """Whole and cut blocks of sixteen rows and columns, one slice and two, runs that begin left of the diagonal or end with the matrix."""
    for d in (1, 2, 3, 15, 16, 17, 31, 34, 63, 64, 67, 129, 260):
        B = inputs.small_int(2900 + N + d, -2, 2, N, d + d % 3).astype(np.float64 if f64 else np.float32)
        want, _ = (oracle.pr_a3_f64 if f64 else oracle.pr_a3)(np.ascontiguousarray(B[:, :d]))
        out = gpu.up(np.full(tet(d), np.nan, dtype=B.dtype))
        (gpu.d.pr_a3_f64 if f64 else gpu.d.pr_a3_f32)(N, d, gpu.up(B), B.shape[1], out)
        assert gpu.down(out).tobytes() == want.astype(B.dtype).tobytes(), d


@pytest.mark.parametrize("N,d", [(1, 40), (15, 97), (16, 97), (40, 33), (64, 150), (64, 260), (100, 256), (128, 257)])
def test_terms_of_few_samples_are_rounded_products(gpu, N, d):
    """One sample that is not zero: the pair rounded, times the third factor within one rounding to nearest (where operands are split, all nine products
    of their parts are added, the smaller eight among themselves: 2^-24 for the last addition, 2^-8 of that for theirs)."""
    B = np.zeros((N, d), dtype=np.float32)
    B[N // 2] = inputs.uniform(3000 + N + d, d)
    out = gpu.empty(tet(d))
    gpu.d.pr_a3_f32(N, d, gpu.up(B), d, out)
    want = expected(B[N // 2])
    assert (np.abs(gpu.down(out).astype(np.float64) - want) <= 2.0 ** -24 * (1 + 2.0 ** -7) * np.abs(want)).all()


WIDE = [(4500, 200, 203), (3001, 257, 257), (1030, 460, 461)]  # staged by more than 15 % of the time that the choice goes by; the last with a workgroup a unit


@pytest.mark.parametrize("N,d,ld", WIDE)
def test_every_part_of_the_split_counts(gpu, N, d, ld):
    """Operands of one bit and of 24, in one sample: a result with one wide operand is exact, whichever of the three it is; with more, the pair is rounded and
    the split leaves out up to 2^-22.4 of a product.  Dropping a third part, or the middle parts' product, would cost 2^-17 of it."""
    b = np.ldexp(1.0, inputs.small_int(3100 + d, -2, 2, d).astype(np.int64)).astype(np.float32)
    wide = np.arange(d) % 3 == 1
    b[wide] = (inputs.uniform(3200 + d, d) + 2.0)[wide].astype(np.float32)
    want = expected(b)
    k = np.arange(d)
    wanted = (k[:, None] <= k[None, :])[:, :, None] & (k[None, :, None] <= k[None, None, :])
    few = (wide.astype(np.int8)[:, None, None] + wide.astype(np.int8)[None, :, None] + wide.astype(np.int8))[wanted] <= 1
    for x in (0, N // 2, N - 1):
        B = np.zeros((N, ld), dtype=np.float32)
        B[x, :d], B[:, d:] = b, np.nan
        out = gpu.empty(tet(d))
        gpu.d.pr_a3_f32(N, d, gpu.up(B), ld, out)
        got = gpu.down(out).astype(np.float64)
        assert np.array_equal(got[few], want[few])
        assert (np.abs(got - want) <= 2.0 ** -22.4 * np.abs(want)).all()


@pytest.mark.parametrize("N,d,ld", WIDE)
def test_staged_sums(gpu, N, d, ld):
    """Slices against products of matrices in double precision.  A term is off by at most 2^-23 (pair) and 2^-22.4 (split), the 16 terms of an instruction are
    added to a sum of n terms with an error of 2^-23 of it: for terms of either sign, sums of n have size sqrt(n) and 2048 at most run together."""
    import torch
    B = gpu.up(inputs.normal(3300 + d, N, ld))
    out = gpu.empty(tet(d))
    gpu.d.pr_a3_f32(N, d, B, ld, out)
    b, run = B[:, :d].double(), min(2048, N)
    bound = 2.0 ** -23 * (2.6 + 4 / 6 * (run / 16) ** 1.5 * (N / run) ** 0.5 / N ** 0.5 * 4)
    for i in (0, 1, d // 2, d - 20):
        want = torch.mm((b * b[:, i:i + 1]).T.contiguous(), b)[i:, i:]
        want = want[torch.triu(torch.ones_like(want, dtype=torch.bool))]
        at = tet(d) - tet(d - i)
        got = out[at:at + len(want)].double()
        assert float((got - want).norm() / want.norm()) < bound


@pytest.mark.parametrize("N,d", [(40, 449), (200, 450), (1030, 460), (2500, 449)])
def test_one_writer_an_element(gpu, N, d):
    """From d = 449 on equal calls give equal bits, also where a workgroup adds up its unit in pieces; a value that is not finite in a later piece."""
    B = inputs.normal(3400 + N, N, d)
    got = []
    for _ in range(3):
        out = gpu.empty(tet(d))
        gpu.d.pr_a3_f32(N, d, gpu.up(B), d, out)
        got.append(gpu.down(out))
    assert got[0].tobytes() == got[1].tobytes() == got[2].tobytes()
    B[N - 3, d - 2] = np.nan
    out = gpu.empty(tet(d))
    gpu.d.pr_a3_f32(N, d, gpu.up(B), d, out)
    k = np.arange(d)
    wanted = (k[:, None] <= k[None, :])[:, :, None] & (k[None, :, None] <= k[None, None, :])
    hit = k == d - 2
    meets = (hit[:, None, None] | hit[None, :, None] | hit)[wanted]
    bad = gpu.down(out)
    assert np.isnan(bad[meets]).all() and np.isfinite(bad[~meets]).all()


@pytest.mark.parametrize("N,d", [(15, 20), (60, 40), (1000, 70)])
@pytest.mark.parametrize("value", [np.nan, np.inf, 1e308])
def test_one_sample_that_is_not_finite_f64(gpu, oracle, N, d, value):
    B = inputs.small_int(3500 + N, 1, 2, N, d).astype(np.float64)
    B[N - 1, d // 2] = value
    with np.errstate(all="ignore"):
        want, _ = oracle.pr_a3_f64(B)
    out = gpu.up(np.full(tet(d), np.nan))
    gpu.d.pr_a3_f64(N, d, gpu.up(B), d, out)
    got, want = gpu.down(out).ravel(), want.ravel()
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))
    ok = np.isfinite(want)
    assert np.allclose(got[ok], want[ok], rtol=2.0 ** -50, atol=0)
