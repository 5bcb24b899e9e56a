"""The gathered transforms' large kernels: every tile width and the odd column counts.

24 atoms of 16 orbitals: the number of vectors moves the tile from 2 to 9
16-column pieces, with widths that do not divide the pairs; 130 occupied states
and ragged rows per atom leave the last tiles of the other side partly empty.
Against the FP64 oracle: FP64 sums in another order, 1e-12 per vector; FP32
transforms, 5e-6.  Odd column counts reach these kernels from a Lanczos
recursion of three drives on a large system only: its coefficients equal the
three single-drive ones (which take the kernels for few columns) to rounding.
"""
import numpy as np
import pytest

from oracle import chi0_oracle as orc

pytestmark = pytest.mark.gpu


def _system(n_atoms, orb, occ, cutoff, cube, placement="whole"):
    from paper_1005_5340_amd import synth
    return synth.make_system(synth.Workload("tiles", n_atoms, orb, occ, 3, 1, cutoff, cube, placement, 0.05, 4, 1.5,
                                            "xyz", 10, 1e-10), 0)


def test_every_tile_width_matches_the_oracle():
    import torch
    from paper_1005_5340_amd import chi0
    s = _system(24, 16, 130, 6.0, 12.0)
    rng = np.random.default_rng(11)
    with chi0.Context(0) as ctx:
        ctx.set_system_from(s)
        for nb in (4, 30, 40, 52, 60, 75, 90, 128):
            om = np.linspace(0.1, 1.2, nb)
            z = rng.standard_normal((nb, s.n_prod)) + 1j * rng.standard_normal((nb, s.n_prod))
            pick = (0, nb // 2, nb - 1)
            ref = {k: orc.chi0_apply(s, float(om[k]), z[k]) for k in pick}
            for precision, tol in ((chi0.PREC_FP64, 1e-12), (chi0.PREC_FP32, 5e-6)):
                out = ctx.apply(om, s.eps, torch.from_numpy(z).cuda(), precision=precision).cpu().numpy()
                for k in pick:
                    assert np.linalg.norm(out[k] - ref[k]) <= tol * np.linalg.norm(ref[k])


def test_odd_column_counts_match_single_drives():
    from paper_1005_5340_amd import chi0
    s = _system(150, 10, 700, 7.0, 20.0, "sequential")
    assert 2.0 * 700 * 3 * 100 * (150 + 2 * np.count_nonzero(s.prod_atoms[:, 1] >= 0)) > 4e8
    d = s.drives("xyz")
    with chi0.Context(0) as ctx:
        ctx.set_system_from(s)
        three = ctx.lanczos(d, k_max=5)
        for q in range(3):
            one = ctx.lanczos(d[q:q + 1], k_max=5)
            for key in ("a", "b"):
                np.testing.assert_allclose(three[key][q], one[key][0], rtol=1e-10)
