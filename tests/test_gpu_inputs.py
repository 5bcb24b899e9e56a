"""How a call's inputs reach the kernels: frequencies as kernel arguments (up to 64)
or by a copy, and the static scratch of the variant without allocation, of which a
call clears only what it reads without having written it.
"""
import numpy as np
import pytest

import gpu_systems

pytestmark = pytest.mark.gpu


def _z(rng, nb, s):
    import torch
    return torch.from_numpy(rng.standard_normal((nb, s.n_prod)) + 1j * rng.standard_normal((nb, s.n_prod))).cuda()


@pytest.mark.parametrize("nb", [1, 63, 64, 65])
def test_every_vector_gets_its_frequency(nb):
    import torch
    from paper_1005_5340_amd import chi0
    s = gpu_systems.get("tiny3")
    rng = np.random.default_rng(2)
    om, z = np.linspace(0.05, 1.4, nb), _z(rng, nb, s)
    with chi0.Context(0) as ctx:
        ctx.set_system_from(s)
        out = ctx.apply(om, s.eps, z)
        for k in (0, nb // 2, nb - 1):
            one = ctx.apply(om[k:k + 1], s.eps, z[k:k + 1])
            assert float(torch.linalg.vector_norm(out[k] - one[0])) <= 1e-12 * float(torch.linalg.vector_norm(one[0]))


@pytest.mark.parametrize("name,nb", [("tiny3", 3), ("atoms12_orb9", 7)])
def test_a_call_after_nan_in_the_scratch_is_clean(name, nb):
    import torch
    from paper_1005_5340_amd import chi0
    s, big = gpu_systems.get(name), gpu_systems.get("atoms12_orb9")
    rng = np.random.default_rng(4)
    om, z = np.linspace(0.1, 1.2, nb), _z(rng, nb, s)
    with chi0.Context(0) as ctx, chi0.Context(0) as other:
        ctx.set_system_from(s)
        other.set_system_from(big)
        ref = ctx.apply(om, s.eps, z)
        bad = torch.full((40, big.n_prod), float("nan"), dtype=torch.complex128, device="cuda")
        assert bool(torch.isnan(other.apply_noalloc(np.full(40, 0.3), big.eps, bad).real).all())
        got = ctx.apply_noalloc(om, s.eps, z)
        assert float(torch.linalg.vector_norm(got - ref)) <= 1e-12 * float(torch.linalg.vector_norm(ref))
