"""FP32 dense transforms at the upper end of the FP32 range.

An operand above 3.39e38 is finite in FP32 but rounds to infinity in BF16, of
which the transforms' three planes are made.  The bound is that of ordinary
operands: three planes hold a value whole, the dropped products are at most 3
2^-25 of |a b| here (the first remainder is up to 2^-8), and each of the 6 K
additions rounds in FP32.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(65, 63, 33), (1000, 3333, 65)])
def test_fp32_operands_up_to_the_largest(M, N, K):
    from paper_1005_5340_amd import chi0
    r = np.random.default_rng(4)
    A = (r.standard_normal((M, K)) * 2.0 ** -12).astype(np.float32).astype(np.float64)
    B = r.uniform(-3.4028234e38, 3.4028234e38, (K, N))
    B[::3] = np.sign(B[::3]) * r.uniform(3.38e38, 3.4028234e38, B[::3].shape)
    B = B.astype(np.float32).astype(np.float64)
    assert np.count_nonzero(np.abs(B) > 3.3961e38) > K * N // 16
    with chi0.Context(0) as ctx:
        got = ctx.debug_panel_gemm(A, B, chi0.PREC_FP32)
    S = np.abs(A) @ np.abs(B)
    assert S.max() < 3e38   # the sums stay in range
    assert np.all(np.abs(got - A @ B) <= (3 * 2.0 ** -25 + 6 * K * 2.0 ** -24) * S)
