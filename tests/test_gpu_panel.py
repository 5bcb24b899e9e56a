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
