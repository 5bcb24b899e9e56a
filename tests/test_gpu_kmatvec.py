"""The skinny kernel product K z at the edges of its dispatch, through the solver.

Two atoms with few orbitals and many products: chi0 has the rank of the few
transitions, so a solve takes a handful of steps at any number of products,
and the residual of its solution, recomputed on the host, shows a wrong
product.  Product counts on both sides of the line between 16- and 32-row
workgroups; 1 to 16 points in flight, i.e. 2 to 32 columns.
"""
import numpy as np
import pytest

from oracle import chi0_oracle as orc

pytestmark = pytest.mark.gpu

TOL = 1e-10


def _system(n_prod):
    from paper_1005_5340_amd import synth
    s = synth.make_system(synth.Workload("pair", 2, 3, 2, n_prod // 2, 0, 4.0, 6.0, "whole", 0.05, 4, 1.5, "z",
                                         10, TOL), 0)
    r = np.random.default_rng(1)
    K = r.standard_normal((s.n_prod, s.n_prod)) * (0.2 / s.n_prod)
    s.K = K + K.T
    s.centroids = r.standard_normal((s.n_prod, 3))
    return s


@pytest.mark.parametrize("n_prod", [60, 5050, 5100])
def test_solutions_meet_the_residual(n_prod):
    from paper_1005_5340_amd import chi0
    s = _system(n_prod)
    d = s.drives("z")
    with chi0.Context(0) as ctx:
        ctx.set_system_from(s)
        for points in (1, 2, 3, 8, 12, 16):
            om = np.linspace(0.1, 1.4, points)
            _, stats, rc, x = ctx.solve_response(om, s.eps, d, restart=20, tol=TOL, batch=points, lanes=1,
                                                 return_x=True)
            assert rc == 0 and np.all(stats["iterations"] >= 1)
            for k, w in enumerate(om):   # the solver met TOL in its own arithmetic: FP64 rounding on top
                assert orc.residual_norm(s, float(w), d[0], x[k, 0], s.eps) <= 2 * TOL
