"""Branches of the dense products that ordinary small systems do not reach.

The INT8 route's ways to cut a column by its length, its largest tiles, its
check; chunks of columns with the frequency factor; the FP64
split-K reduction with the factor; the tile variants of the FP64 GEMM, split
and whole.  References in extended precision or the FP64 oracle.
"""
import numpy as np
import pytest

from oracle import chi0_oracle as orc

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def ctx():
    from paper_1005_5340_amd import chi0
    with chi0.Context(0) as c:
        yield c


def _operands(M, N, K, seed):
    r = np.random.default_rng(seed)
    A = r.standard_normal((M, K)) * np.exp2(r.integers(-6, 7, (M, 1)))
    B = r.standard_normal((K, N)) * np.exp2(r.integers(-20, 21, (1, N)))
    return A, B


def _check_rows(got, A, B, rows):
    """Every element within the bound of an FP64 sum."""
    A = A[rows].astype(np.longdouble)
    S = np.abs(A) @ np.abs(B)
    assert np.all(np.abs(got[rows] - A @ B.astype(np.longdouble)) <= A.shape[1] * np.longdouble(U) * S)


@pytest.mark.parametrize("M,N,K", [(64, 40, 1024), (64, 40, 1500), (64, 40, 2049), (64, 40, 4096), (64, 40, 4100),
                                   (64, 40, 6144), (64, 40, 6145), (64, 300, 7000), (256, 300, 1024), (256, 300, 1040),
                                   (512, 257, 5200)])
def test_int8_route_by_length(ctx, M, N, K):
    """A column of up to 1024, 2048, 4096 and 6144 entries is cut by one workgroup, a longer one by two
    kernels; 256-row tiles from K = 1024, with stages of 8 or 4 blocks of 16."""
    from paper_1005_5340_amd import chi0
    A, B = _operands(M, N, K, 21)
    B[K // 2, ::7] *= 2.0 ** 45       # columns for the FP64 tiles ...
    A[1::2, K // 2] = 0.0
    B[:, -40:-1] = B[:, :39] * 2.0 ** -3
    got, tiles = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
    assert tiles > 0
    rows = np.r_[0:min(M, 64), max(M - 64, 64):M]
    _check_rows(got, A, B, rows)
    A, B = _operands(M, N, K, 22)     # ... and none
    got, tiles = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
    assert tiles == 0
    _check_rows(got, A, B, rows)


@pytest.mark.parametrize("K", [64, 128])
def test_check_of_large_products(ctx, K):
    """Many tiles, of which one goes to FP64."""
    from paper_1005_5340_amd import chi0
    M, N = 1024, 8192
    A, B = _operands(M, N, K, 23)
    A[512:576, 3] = 0.0               # one tile of 64 x 128: rows 512.. and columns 4096..
    B[3, 4096:4224] *= 2.0 ** 45
    got, tiles = ctx.debug_dense_transform(A, B, chi0.PREC_FP64)
    assert 1 <= tiles < M // 64 * (N // 128)
    _check_rows(got, A, B, np.r_[500:520, 570:580, 0, M - 1])


def _factor(N, M, nb, seed):
    r = np.random.default_rng(seed)
    om = np.linspace(0.2, 1.3, nb)
    D = r.uniform(0.3, 2.0, (N // (2 * nb), M))
    eps = 0.01
    L = np.array([[2.0 / (w - D + 1j * eps) - 2.0 / (w + D + 1j * eps) for w in om]])[0]   # [nb, E, M]
    return om, D, eps, L


def _with_factor(P, L, nb):
    """P [M, N] -> complex [M, E, nb], times the factor."""
    M, N = P.shape
    c = P.reshape(M, N // (2 * nb), nb, 2)
    return (c[..., 0] + 1j * c[..., 1]) * np.transpose(L, (2, 1, 0))


# the error of the product K u S (FP64), of its dropped terms and FP32 additions (the others), in both parts,
# times |L|; the factor and the result round some 40 times in FP64, the operands and the result once in FP32
@pytest.mark.parametrize("precision,M,N,K", [("fp64", 128, 1500, 100), ("fp64", 192, 3000, 410), ("fp32", 256, 8400, 40),
                                             ("bf16x3", 256, 8400, 40), ("fp32", 64, 600, 300)])
def test_chunks_of_columns_with_the_factor(ctx, precision, M, N, K):
    from paper_1005_5340_amd import chi0
    nb, prec = 3, dict(fp64=chi0.PREC_FP64, fp32=chi0.PREC_FP32, bf16x3=chi0.PREC_BF16X3)[precision]
    A, B = _operands(M, N, K, 31)
    if precision == "fp64":           # some tiles of some chunks go to the FP64 matrix cores
        A[5, 7] = 0.0
        B[7, 700:720] *= 2.0 ** 45
    else:
        A, B = A.astype(np.float32).astype(float), B.astype(np.float32).astype(float)
    om, D, eps, L = _factor(N, M, nb, 32)
    whole, t1 = ctx.debug_dense_transform(A, B, prec, 1 << 30, om, eps, 2.0, D)
    parts, t2 = ctx.debug_dense_transform(A, B, prec, 0, om, eps, 2.0, D)
    assert np.array_equal(whole, parts) and t1 == t2 and (t1 > 0) == (precision == "fp64")
    S = np.abs(A) @ np.abs(B)
    S = S.reshape(M, -1, nb, 2).sum(-1)
    rel = {"fp64": K * U, "fp32": 3 * 2.0 ** -27 + 6 * K * 2.0 ** -24, "bf16x3": 3 * 2.0 ** -18 + 3 * K * 2.0 ** -24}
    rnd = 40 * U if precision == "fp64" else 2.0 ** -23
    ref = _with_factor((A.astype(np.longdouble) @ B.astype(np.longdouble)).astype(float) if precision == "fp64" else A @ B,
                       L, nb)
    got = parts.reshape(M, -1, nb, 2)
    got = got[..., 0] + 1j * got[..., 1]
    absL = np.abs(np.transpose(L, (2, 1, 0)))
    # (the reference's own factor cancels near D = 0 by a few roundings of 1 / D^2: within rnd of |L| S)
    assert np.all(np.abs(got - ref) <= absL * S * (rel[precision] + rnd) * (1 + 1e-6) + rnd * np.abs(ref))


def _workload(name, n_atoms, orb, occ, per_atom, per_pair):
    from paper_1005_5340_amd import synth
    return synth.make_system(synth.Workload(name, n_atoms, orb, occ, per_atom, per_pair, 5.0,
                                            (25.0 * n_atoms) ** (1 / 3), "sequential", 0.01, 4, 1.5, "z", 10, 1e-10), 0)


def test_split_k_with_the_factor_matches_the_oracle():
    """Few occupied states and many orbitals: large products of few columns, whose sums are split over
    workgroups and put together, with the factor, by the reduction (the last part runs over the padding)."""
    import torch
    from paper_1005_5340_amd import chi0
    s = _workload("split", 100, 13, 16, 2, 1)
    nb = 15
    assert 1344 * 16 * 2 * nb * 1296 > 8e8 and 1344 // 64 * (16 * 2 * nb // 64 + 1) < 256
    r = np.random.default_rng(9)
    om = np.linspace(0.1, 1.2, nb)
    z = r.standard_normal((nb, s.n_prod)) + 1j * r.standard_normal((nb, s.n_prod))
    zt = torch.from_numpy(z).cuda()
    with chi0.Context(0) as c:
        c.set_system_from(s)
        c.apply(om, s.eps, zt)
        c.set_timing(True)
        out = c.apply(om, s.eps, zt).cpu().numpy()
        st = c.kernel_stats()
    assert st["splitk_reduce"]["launches"] == 2 and st["virt_transform_lorentz"]["launches"] == 1
    for k, w in enumerate(om):
        ref = orc.chi0_apply(s, float(w), z[k])
        assert np.linalg.norm(out[k] - ref) <= 1e-12 * np.linalg.norm(ref)


def test_every_tile_variant_on_whole_and_split_sums():
    """The six tile variants forced in turn where all of them are valid (row counts that are multiples of
    128, sums of multiples of 32): the operator, whose sums are whole, and a batch of solver steps, whose
    K V is split, equal the first variant's bit for bit."""
    import torch
    from paper_1005_5340_amd import chi0, synth
    s = _workload("variants", 40, 12, 100, 2, 1)          # 512 x 384 padded
    nb = 24
    assert 384 * 112 * 2 * nb * 480 > 8e8
    s60 = synth.make_system("atoms60_orb9", 0)            # 3328 products padded
    om60 = np.linspace(0.05, 1.4, 40)
    assert -(-s60.n_prod // 64) * 64 == 3328 and 3328 ** 2 * 80 > 8e8
    r = np.random.default_rng(12)
    om = np.linspace(0.1, 1.2, nb)
    z = torch.from_numpy(r.standard_normal((nb, s.n_prod)) + 1j * r.standard_normal((nb, s.n_prod))).cuda()
    first = None
    for v in range(6):
        with chi0.Context(0) as c, chi0.Context(0) as c60:
            c.set_system_from(s)
            c60.set_system_from(s60)
            c.set_autotune(False, force_variant=v)
            c60.set_autotune(False, force_variant=v)
            c.set_timing(True)
            c60.set_timing(True)
            out = c.apply(om, s.eps, z).cpu().numpy()
            a, st, rc = c60.solve_response(om60, s60.eps, s60.drives("z"), restart=s60.n_prod, tol=1e-2, batch=40, lanes=1)
            assert rc == 0
            st, st60 = c.kernel_stats(), c60.kernel_stats()
            assert "splitk_reduce" not in st or st["splitk_reduce"]["launches"] == 0
            assert st["virt_transform_lorentz"]["launches"] == 1 and st["virt_back"]["launches"] == 1
            assert st60["kernel_matmul"]["launches"] >= 3 and st60["splitk_reduce"]["launches"] >= 3
        if first is None:
            first = out, a
        assert np.array_equal(out, first[0]), f"variant {v} changed chi0 z"
        assert np.array_equal(a, first[1]), f"variant {v} changed the solve"


def test_graph_replays_of_the_int8_route():
    """Replays with other vectors in the same buffer, of which some have tiles for the FP64 matrix cores
    and some none, equal eager calls bit for bit, with eager work and synchronisations in between."""
    import torch
    from paper_1005_5340_amd import chi0
    s = _workload("replay", 120, 10, 500, 2, 1)
    r = np.random.default_rng(17)
    om = np.array([0.3, 0.8])
    z = torch.zeros((2, s.n_prod), dtype=torch.complex128, device="cuda")
    out = torch.empty_like(z)
    with chi0.Context(0) as ca, chi0.Context(0) as cb:
        ca.set_system_from(s)
        cb.set_system_from(s)
        ca.set_graphs(True)
        cb.set_timing(True)
        for rep in range(7):
            zh = r.standard_normal((2, s.n_prod)) + 1j * r.standard_normal((2, s.n_prod))
            if rep % 3 == 2:
                zh[1] *= np.exp2(r.integers(-200, 0, s.n_prod))
            if rep == 5:
                zh[0] = 0.0
                zh[0, 4] = 1.0
            z.copy_(torch.from_numpy(zh))
            ca.apply(om, s.eps, z, out=out)
            ref = cb.apply(om, s.eps, z.clone())
            torch.cuda.synchronize()
            assert torch.equal(out, ref), rep
        assert cb.kernel_stats()["virt_back_crt"]["launches"] == 7
