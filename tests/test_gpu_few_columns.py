"""The transforms for few columns at the edges of their splits.

Three atoms whose pairs all overlap, so a call is small whatever the sizes:
the gathered transforms split the gathered rows (32 or 64 per round of a
workgroup's waves) or the occupied states, and cut an atom's (orbital, column)
pairs into tiles of 16 that begin and end inside one orbital; the dense ones
split k and take 16 x 16 tiles, 32 x 32 above 2^17 outputs.  Against the FP64
oracle: FP64 sums in another order, 1e-12 per vector; FP32 transforms, 5e-6.
"""
import numpy as np
import pytest

from oracle import chi0_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("orb,occ,nb", [(1, 1, 1), (3, 2, 1), (5, 7, 3), (11, 17, 2), (11, 16, 9), (16, 33, 1),
                                        (16, 32, 33), (13, 5, 50), (16, 31, 70)])
def test_few_columns_match_the_oracle(orb, occ, nb):
    import torch
    from paper_1005_5340_amd import chi0, synth
    s = synth.make_system(synth.Workload("few", 3, orb, occ, 3, 2, 9.0, 4.0, "whole", 0.05, 4, 1.5, "z", 10, 1e-10), 0)
    rng = np.random.default_rng(7)
    om = np.linspace(0.1, 1.2, nb)
    z = rng.standard_normal((nb, s.n_prod)) + 1j * rng.standard_normal((nb, s.n_prod))
    ref = [orc.chi0_apply(s, float(w), z[k]) for k, w in enumerate(om)]
    with chi0.Context(0) as ctx:
        ctx.set_system_from(s)
        for precision, tol in ((chi0.PREC_FP64, 1e-12), (chi0.PREC_FP32, 5e-6)):
            out = ctx.apply(om, s.eps, torch.from_numpy(z).cuda(), precision=precision).cpu().numpy()
            for k in range(nb):
                assert np.linalg.norm(out[k] - ref[k]) <= tol * np.linalg.norm(ref[k])
