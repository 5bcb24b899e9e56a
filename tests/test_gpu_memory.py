"""A nearly full device: what the INT8 route holds gives way.

The residues of the orbitals and the workspaces that go with them only make a
call faster.  With less memory than they want (a limit that a test hook sets
stands for the full device) every call that needs none of them still runs and
gives the same answer: FP64 sums in another order, 1e-12 per vector; chunks of
columns change no sum of the FP32 transforms, nor does the recursion use them.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    import torch
    from paper_1005_5340_amd import chi0, synth
    s = synth.make_system(synth.Workload("memory", 150, 10, 640, 2, 1, 5.0, 3750.0 ** (1 / 3), "sequential", 0.01, 4,
                                         1.5, "z", 10, 1e-10), 0)
    r = np.random.default_rng(3)
    om = np.array([0.2, 0.6, 1.1])
    z = torch.from_numpy(r.standard_normal((3, s.n_prod)) + 1j * r.standard_normal((3, s.n_prod))).cuda()
    with chi0.Context(0) as c:
        c.set_system_from(s)
        out = c.apply(om, s.eps, z)
        held, optional = c.debug_memory()
        assert optional > 0
        f32 = c.apply(om, s.eps, z, precision=chi0.PREC_FP32)
        lz = c.lanczos(s.drives("z"), k_max=5)
    return s, om, z, out, f32, lz, held, optional


def _same(a, b):
    import torch
    return float((torch.linalg.vector_norm(a - b, dim=1) / torch.linalg.vector_norm(b, dim=1)).max()) <= 1e-12


@pytest.mark.parametrize("part", [0.0, 0.25, 0.6, 0.999])
def test_apply_with_part_of_the_optional_memory(case, part):
    from paper_1005_5340_amd import chi0
    s, om, z, out, _, _, held, optional = case
    limit = held - optional + int(part * optional)
    with chi0.Context(0) as c:
        c.debug_memory(limit)
        c.set_system_from(s)
        assert _same(c.apply(om, s.eps, z), out)
        got, opt = c.debug_memory(limit)
        print(f"[memory] limit {limit}: held {got}, optional {opt}", flush=True)
        assert got <= limit and (opt > 0) == (part > 0.0)


def test_other_allocations_take_it_back(case):
    import torch
    from paper_1005_5340_amd import chi0
    s, om, z, out, f32, lz, held, optional = case
    with chi0.Context(0) as c:
        c.set_system_from(s)
        c.apply(om, s.eps, z)
        assert c.debug_memory(held) == (held, optional)   # nothing more from here on
        got = c.lanczos(s.drives("z"), k_max=5)
        assert np.array_equal(got["a"], lz["a"]) and np.array_equal(got["b"], lz["b"])
        assert c.debug_memory(held)[1] < optional
        assert torch.equal(c.apply(om, s.eps, z, precision=chi0.PREC_FP32), f32)
        assert _same(c.apply(om, s.eps, z), out)
        # and an allocation that does not fit even so is refused, with the context still good
        c.debug_memory(c.debug_memory(held)[0] - c.debug_memory(held)[1])
        with pytest.raises(chi0.Chi0Error) as e:
            c.lanczos(s.drives("z"), k_max=5)
        assert e.value.code == -3
        c.debug_memory(-1)
        assert _same(c.apply(om, s.eps, z), out)


def test_solver_lanes_share_what_is_left(case):
    """Two lanes, each with a workspace of its own, where only part of the INT8 route's memory is there:
    the solutions meet the same tolerance."""
    from paper_1005_5340_amd import chi0
    s, om, z, out, _, _, _, _ = case
    d = s.drives("z")
    grid = np.linspace(0.4, 1.2, 16)

    def solve(limit):
        with chi0.Context(0) as c:
            c.debug_memory(limit)
            c.set_system_from(s)
            a, st, rc = c.solve_response(grid, s.eps, d, restart=200, tol=1e-10, batch=16, lanes=2)
            assert rc == 0
            return a, c.debug_memory(limit)

    ref, (held, optional) = solve(-1)
    assert optional > 0
    call = 1 << 20   # more than what a call takes and gives back
    for part in (0.0, 0.3, 0.8):
        got, (h, o) = solve(held - optional + call + int(part * optional))
        print(f"[memory] lanes, part {part}: held {h}, optional {o}", flush=True)
        assert h <= held - (1.0 - part) * optional + call
        # both meet a residual of 1e-10; the polarizability is second-order accurate in it
        assert np.max(np.abs(got - ref)) <= 1e-9 * np.max(np.abs(ref))
