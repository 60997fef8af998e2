"""GPU: postponed solution updates (a ring of corrections added to u later) are
bit for bit updates in place."""
import pytest
import torch

from paper_2007_07539_amd import mgir
from paper_2007_07539_amd import workloads as W

pytestmark = pytest.mark.gpu


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
