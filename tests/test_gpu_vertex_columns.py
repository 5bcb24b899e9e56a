"""The vertex kernels for few columns at the edges of their splits.

Up to 16 columns a workgroup of the gather splits the products of a block over
its wavefronts when there are more than 32, in two row groups up to 128 rows
and four above, and one of the projection splits the rows; the results leave
in groups of 8 vectors.  Products per block and rows on both sides of each
line, 1 to 9 vectors (2 to 18 columns), against the FP64 oracle; FP64 sums in
another order, so 1e-12 per vector as for every size.
"""
import numpy as np
import pytest

from oracle import chi0_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("orb,per_atom,per_pair", [(3, 4, 1), (11, 28, 2), (12, 30, 3), (11, 29, 2), (16, 90, 17),
                                                   (5, 260, 40)])
def test_few_columns_match_the_oracle(orb, per_atom, per_pair):
    import torch
    from paper_1005_5340_amd import chi0, synth
    s = synth.make_system(synth.Workload("few", 3, orb, 2, per_atom, per_pair, 9.0, 4.0, "whole", 0.05, 4, 1.5, "z",
                                         10, 1e-10), 0)
    assert len(s.prod_atoms) == 3 * per_atom + 3 * per_pair   # every pair overlaps
    rng = np.random.default_rng(5)
    with chi0.Context(0) as ctx:
        ctx.set_system_from(s)
        for nb in (1, 3, 8, 9):
            om = np.linspace(0.1, 1.2, nb)
            z = rng.standard_normal((nb, s.n_prod)) + 1j * rng.standard_normal((nb, s.n_prod))
            out = ctx.apply(om, s.eps, torch.from_numpy(z).cuda()).cpu().numpy()
            for k, w in enumerate(om):
                ref = orc.chi0_apply(s, float(w), z[k])
                assert np.linalg.norm(out[k] - ref) <= 1e-12 * np.linalg.norm(ref)
