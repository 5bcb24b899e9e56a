"""The panel GEMMs of the dense transforms against the product in extended precision.

Sizes: below one tile, at the edges of the 64- and 128-row and -column tiles
and one past them, reduction lengths below, at and past one stage, a product
large enough for the 128 x 128 tiles, and column chunks with a ragged last one.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1005_5340_amd import chi0
    with chi0.Context(0) as c:
        yield c


SIZES = [(1, 1, 1), (64, 64, 32), (65, 63, 33), (128, 130, 31), (300, 17, 540), (129, 1000, 96),
         (200, 257, 1031), (1000, 3333, 65)]


def _operands(M, N, K, seed):
    r = np.random.default_rng(seed)
    # columns and rows of very different sizes, as the response vectors have
    A = r.standard_normal((M, K)) * np.exp2(r.integers(-6, 7, (M, 1)))
    B = r.standard_normal((K, N)) * np.exp2(r.integers(-20, 21, (1, N)))
    return A, B


@pytest.mark.parametrize("M,N,K", SIZES)
@pytest.mark.parametrize("chunk", [0, 1 << 30])
def test_bf16x3(ctx, M, N, K, chunk):
    """x = hi + lo + e with |lo| <= 2^-9 |x| and |e| <= 2^-18 |x|: the dropped parts of a product are
    at most 3 2^-18 |a b|, and each of its 3 K additions rounds in FP32 (the inputs are rounded to it)."""
    from paper_1005_5340_amd import chi0
    A, B = _operands(M, N, K, 1)
    got = ctx.debug_panel_gemm(A, B, chi0.PREC_BF16X3, chunk)
    A, B = A.astype(np.float32).astype(np.float64), B.astype(np.float32).astype(np.float64)
    bound = (3 * 2.0 ** -18 + 3 * K * 2.0 ** -24) * (np.abs(A) @ np.abs(B))
    assert np.all(np.abs(got - A @ B) <= bound)


@pytest.mark.parametrize("M,N,K", SIZES)
@pytest.mark.parametrize("chunk", [0, 1 << 30])
def test_fp32(ctx, M, N, K, chunk):
    """Three planes hold an FP32 value whole, |plane i| <= 2^-9i |x|: the dropped products are at most
    2 2^-27 + 2^-36 of |a b|, and each of its 6 K additions rounds in FP32."""
    from paper_1005_5340_amd import chi0
    A, B = _operands(M, N, K, 2)
    got = ctx.debug_panel_gemm(A, B, chi0.PREC_FP32, chunk)
    A, B = A.astype(np.float32).astype(np.float64), B.astype(np.float32).astype(np.float64)
    bound = (3 * 2.0 ** -27 + 6 * K * 2.0 ** -24) * (np.abs(A) @ np.abs(B))
    assert np.all(np.abs(got - A @ B) <= bound)


def _product_longdouble(A, B):
    return A.astype(np.longdouble) @ B.astype(np.longdouble)


@pytest.mark.parametrize("M,N,K", [(-(-m // 4) * 4, n, k) for m, n, k in SIZES])
@pytest.mark.parametrize("chunk", [0, 1 << 30])
def test_fp64_on_int8(ctx, M, N, K, chunk):
    """Entries are rounded to at most 2^-54.5 of their row's or column's norm and no finer than 2^-53.9
    of its largest entry (each half a unit off), so a sum of K products is off by at most
    sqrt(K) 2^-52.8 |A_i| |B_j|; putting it together and scaling it round seven times (2^-50 |C|)."""
    from paper_1005_5340_amd import chi0
    A, B = _operands(M, N, K, 3)
    B[:, N // 2] = 0.0
    got = ctx.debug_panel_gemm(A, B, chi0.PREC_FP64, chunk)
    ref = _product_longdouble(A, B)
    norms = np.linalg.norm(A, axis=1)[:, None] * np.linalg.norm(B, axis=0)[None, :]
    bound = np.sqrt(K) * 2.0 ** -52.8 * norms + 2.0 ** -50 * np.abs(ref)
    assert np.all(np.abs(got - ref) <= bound)
    # and as a whole no worse than the FP64 product that it stands in for
    assert np.linalg.norm((got - ref).astype(float)) <= 1e-15 * np.sqrt(max(K, 16) / 16) * np.linalg.norm(norms)


def test_fp64_on_int8_extremes(ctx):
    """Entries far below or beyond the usual range keep their relative accuracy; a column with an
    infinity or NaN is NaN and leaves the others alone."""
    from paper_1005_5340_amd import chi0
    r = np.random.default_rng(5)
    M, N, K = 68, 300, 129
    B = r.standard_normal((K, N))
    B[:, 0] *= 1e-300
    B[:, 1] *= 1e300
    B[:, 2] *= 1e-310          # subnormal: rounded to 2^-1074 on input already
    B[:, 3] = 0.0
    B[5, 3] = 1e-200           # one entry alone
    B[7, 4] = np.inf
    B[8, 5] = np.nan
    A = r.standard_normal((M, K)) * 1e-2
    got = ctx.debug_panel_gemm(A, B, chi0.PREC_FP64)
    assert np.all(np.isnan(got[:, 4:6])) and np.all(np.isfinite(np.delete(got, [4, 5], axis=1)))
    ref = _product_longdouble(A, B[:, [0, 1, 2, 3, 6]])
    norms = np.linalg.norm(A, axis=1)[:, None] * np.sqrt((B[:, [0, 1, 2, 3, 6]].astype(np.longdouble) ** 2).sum(0))
    tiny = np.longdouble(2.0) ** -1074
    assert np.all(np.abs(got[:, [0, 1, 2, 3, 6]] - ref) <= np.sqrt(K) * 2.0 ** -52.8 * norms
                  + 2.0 ** -50 * np.abs(ref) + tiny)
