"""FP64 dense transforms whose operands span a wide range inside a row or column.

On the INT8 matrix cores a column is rounded on one scale, so an element of the
product whose own terms are small against the norms (large entries of one
operand meet zeros or small ones of the other) is only right if its tile goes
to the FP64 matrix cores.  Every element has to meet the bound of an FP64 sum,
K 2^-53 sum_k |A_ik| |B_kj|, the check's own criterion (which leaves room for
the roundings of the scaling); the reference is in extended precision, and the
tiny absolute term is that of subnormal results.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1005_5340_amd import chi0
    with chi0.Context(0) as c:
        yield c


def _operands(kind, M, N, K, seed):
    r = np.random.default_rng(seed)
    A, B = r.standard_normal((M, K)), r.standard_normal((K, N))
    if kind == "zeros meet large entries":       # ten of one row, in every column
        k = r.choice(K, 10, replace=False)
        A[M // 2, k] = 0.0
        B[k] *= 2.0 ** 30
    elif kind == "one column":                   # the rest of the tile is ordinary
        A[7, :5] = 0.0
        B[:5, N // 3] *= 2.0 ** 40
    elif kind == "graded":
        B *= np.exp2(r.integers(-40, 41, (K, N)))
        A *= np.exp2(r.integers(-10, 11, (M, K)))
    elif kind == "two classes":                  # exact zeros by symmetry
        A[:M // 2, K // 2:] = 0.0
        A[M // 2:, :K // 2] = 0.0
        B[:K // 2] *= 2.0 ** 30
    elif kind == "two classes, nearly":          # the same zeros with rounding noise in them
        A[:M // 2, K // 2:] *= 2.0 ** -53
        A[M // 2:, :K // 2] *= 2.0 ** -53
        B[:K // 2] *= 2.0 ** 30
    elif kind == "one entry":                    # columns and rows with a single entry, far from one
        B[:, ::3] = 0.0
        B[5, ::3] = 1e-200
        A[::5] = 0.0
        A[::5, 5] = 1e-30
    elif kind == "tiny and large columns":
        B *= np.exp2(r.integers(-900, 901, (1, N)))
        B[3] *= 2.0 ** -60
        A[:, 4] = 0.0
        B[4] *= 2.0 ** 35
    return A, B


def _product_longdouble(A, B):
    return A.astype(np.longdouble) @ B.astype(np.longdouble)


@pytest.mark.parametrize("M,N,K", [(64, 20, 96), (192, 300, 515)])
@pytest.mark.parametrize("kind", ["zeros meet large entries", "one column", "graded", "two classes",
                                  "two classes, nearly", "one entry", "tiny and large columns"])
def test_every_element_keeps_the_bound_of_an_fp64_sum(ctx, kind, M, N, K):
    from paper_1005_5340_amd import chi0
    A, B = _operands(kind, M, N, K, 11)
    got, tiles = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
    ref, S = _product_longdouble(A, B), _product_longdouble(np.abs(A), np.abs(B))
    print(f"[range] {kind} {M}x{N}x{K}: {tiles} tiles in FP64", flush=True)
    assert np.all(np.abs(got - ref) <= K * np.longdouble(2.0) ** -53 * S + np.longdouble(2.0) ** -1070)


@pytest.mark.parametrize("M,N,K", [(64, 64, 290), (320, 700, 544), (192, 300, 1030)])
def test_ordinary_operands_stay_on_int8(ctx, M, N, K):
    """Dense operands, rows and columns of any size, padding rows and columns, also a response with a
    transition 2 eps from resonance (a factor of about 50), the shortest sums below those that the dispatch
    sends here: no tile leaves."""
    from paper_1005_5340_amd import chi0
    r = np.random.default_rng(3)
    A = r.standard_normal((M, K)) * np.exp2(r.integers(-6, 7, (M, 1)))
    B = r.standard_normal((K, N)) * np.exp2(r.integers(-20, 21, (1, N)))
    B[r.integers(0, K, N), np.arange(N)] *= 50.0
    A[-3:] = 0.0
    B[:, N // 2] = 0.0
    got, tiles = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
    assert tiles == 0
    ref = _product_longdouble(A, B)
    assert np.all(np.abs(got - ref) <= K * 2.0 ** -53 * _product_longdouble(np.abs(A), np.abs(B)))
    # exact zeros by symmetry alone are no reason to leave: those elements come out as zeros
    A[:32, K // 2:] = 0.0
    B[:K // 2, :32] = 0.0
    got, tiles = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
    assert tiles == 0 and np.all(got[:32, :32] == 0.0)


def test_infinities_and_nan_as_in_an_fp64_sum(ctx):
    from paper_1005_5340_amd import chi0
    r = np.random.default_rng(5)
    A, B = r.standard_normal((128, 200)), r.standard_normal((200, 300))
    B[7, 4] = np.inf
    B[8, 5] = np.nan
    B[9, 290] = -np.inf
    got, _ = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
    with np.errstate(invalid="ignore"):
        ref = A @ B
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    fin = np.isfinite(ref)
    assert np.all(got[~fin & ~np.isnan(ref)] == ref[~fin & ~np.isnan(ref)])
    assert np.allclose(got[fin], ref[fin], rtol=0, atol=1e-11)


def _two_class_system():
    """Even and odd orbitals of every atom do not mix; odd products couple the two classes, even ones do not."""
    from paper_1005_5340_amd import synth
    s = synth.make_system(synth.Workload("classes", 100, 13, 640, 2, 2, 5.0, 2500.0 ** (1 / 3), "sequential",
                                         0.01, 4, 1.5, "z", 10, 1e-10), 0)
    r = np.random.default_rng(2)
    n = s.n_orb
    cls = np.tile(np.arange(13) % 2, 100)
    X = np.zeros((n, n))
    # the states of a class are spread evenly over occupied and virtual ones
    where = np.argsort(np.concatenate([(np.arange(c) + 0.5) / c for c in (np.sum(cls == 0), np.sum(cls == 1))]),
                       kind="stable")
    start = 0
    for q in (0, 1):
        idx = np.nonzero(cls == q)[0]
        cols = np.nonzero((where >= start) & (where < start + idx.size))[0]
        X[np.ix_(idx, cols)] = np.linalg.qr(r.standard_normal((idx.size, idx.size)))[0]
        start += idx.size
    s.X = X
    vb = s.vblock.copy()
    for mu in range(s.n_prod):
        c = cls[s.support(mu)]
        o = int(s.vblock_offset[mu])
        same = c[:, None] == c[None, :]
        vb[o:o + c.size ** 2].reshape(c.size, c.size)[same == bool(mu % 2)] = 0.0
    s.vblock = vb
    return s


def test_small_part_of_a_response_next_to_a_large_one():
    """chi0 z of a vector whose coupling part is 2^-30 of the other: the coupling products' response is that
    of the coupling part alone, by symmetry, and right to the 1e-12 that an FP64 sum gives."""
    import torch
    from oracle import chi0_oracle as orc
    from paper_1005_5340_amd import chi0
    s = _two_class_system()
    r = np.random.default_rng(7)
    om = np.array([0.3, 0.7, 1.1])
    z = r.standard_normal((3, s.n_prod)) + 1j * r.standard_normal((3, s.n_prod))
    small = np.arange(s.n_prod) % 2 == 1
    z[:, small] *= 2.0 ** -30
    with chi0.Context(0) as c:
        c.set_system_from(s)
        c.set_timing(True)
        out = c.apply(om, s.eps, torch.from_numpy(z).cuda()).cpu().numpy()
        st = c.kernel_stats()
        assert st["virt_transform_crt"]["launches"] == 1 and st["virt_back_crt"]["launches"] == 1
    for k, w in enumerate(om):
        ref = orc.chi0_apply(s, float(w), z[k])
        for part in (small, ~small):
            e = np.linalg.norm(out[k, part] - ref[part]) / np.linalg.norm(ref[part])
            print(f"[range] omega {w} {'coupling' if part is small else 'other'} products: {e:.2e}", flush=True)
            assert e <= 1e-12


@pytest.mark.parametrize("M,N,K", [(64, 64, 900), (64, 64, 1000), (128, 200, 460), (1024, 8192, 100), (1024, 8192, 120)])
def test_operands_that_meet_in_one_block_only(ctx, M, N, K):
    """One row and one column of ordinary matrices share a single block of 16 terms, 2^-40 of their others,
    which meet zeros: the check has to look at every block."""
    from paper_1005_5340_amd import chi0
    r = np.random.default_rng(13)
    blk = np.arange(K) // 16
    A0, B0 = r.standard_normal((M, K)), r.standard_normal((K, N))
    for b in range(-(-K // 16)):
        A, B = A0.copy(), B0.copy()
        A[3] *= np.where(blk == b, 2.0 ** -40, blk % 2 == 0)
        B[:, 5] *= np.where(blk == b, 2.0 ** -40, blk % 2 == 1)
        got, tiles = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
        ref, S = _product_longdouble(A[3:4], B), _product_longdouble(np.abs(A[3:4]), np.abs(B))
        assert tiles > 0 and np.all(np.abs(got[3] - ref) <= K * np.longdouble(2.0) ** -53 * S), b
