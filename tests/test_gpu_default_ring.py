"""GPU: large grids postpone their solution updates by default (a ring of eight
corrections); u is bit for bit that of updating in place, over a full ring and a
remainder, from zero and from a guess, on repeated solves."""
import pytest
import torch

from paper_2007_07539_amd import mgir
from paper_2007_07539_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n,name,disc", [(3, 255, "f16", "fd"), (3, 255, "f32", "fd"), (2, 2303, "f16", "q1")])
def test_default_ring_is_bitwise(dim, n, name, disc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    prec = W.precision_map(name, mgir.full_levels(n))
    g = torch.Generator(device="cuda").manual_seed(n)
    b = torch.rand((n,) * dim, dtype=torch.float64, device="cuda", generator=g) - 0.5
    if disc == "q1":
        b = b / float(n + 1) ** dim
    u0 = torch.rand((n,) * dim, dtype=torch.float64, device="cuda", generator=g)
    for guess in (False, True):
        print(f"default ring {dim}-D n={n} {name} {disc} guess={guess}", flush=True)
        kw = dict(disc=disc, max_iter=10, rtol=0.0, use_initial_guess=guess)
        s = mgir.Solver(dim, n, prec, **kw)
        assert "defer_flush" in [r[0] for r in s.profile_step()]
        if disc == "fd":
            ref = mgir.Solver(dim, n, prec, **kw)
            ref.set_shape(0, mgir.SHAPE_FUSE, [0])  # u updated in place
            assert "defer_flush" not in [r[0] for r in ref.profile_step()]
        else:
            ref = mgir.Solver(dim, n, prec, defer_update=1, **kw)  # added to u in every step
        want = ref.solve(b, u0.clone(), check=False)[0]
        for _ in range(2):
            assert torch.equal(s.solve(b, u0.clone(), check=False)[0], want)


def test_ring_unused_without_the_fused_update():
    """A ring that the fused update would fill is not used once that kernel is switched off: u starts
    from zero and is updated in place (it used to start from whatever the last solve had left)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("ring without the fused update", flush=True)
    n = 31
    prec = W.precision_map("f16", mgir.full_levels(n))
    g = torch.Generator(device="cuda").manual_seed(3)
    b = torch.rand((n,) * 3, dtype=torch.float64, device="cuda", generator=g) - 0.5
    want = mgir.Solver(3, n, prec).solve(b)[0].clone()
    s = mgir.Solver(3, n, prec, defer_update=4)
    s.set_shape(0, mgir.SHAPE_FUSE, [0])
    for _ in range(2):
        assert torch.equal(s.solve(b)[0], want)
