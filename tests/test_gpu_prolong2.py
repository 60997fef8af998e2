"""GPU: the prolongation fused with two post-sweeps, on every pitch it serves
(one tile, several, a ragged last one) and pair of formats, with two and three
post-sweeps, as the cycle's finest level and below it.  Same roundings as the
separate kernels (which the level takes once a shape of its sweep is set), so
every V-cycle is equal bit for bit."""
import pytest
import torch

from paper_2007_07539_amd import mgir

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", [["f16"], ["bf16", "f32", "f16"], ["f32", "f64", "bf16"], ["f64", "f16", "f64"],
                                 ["f16", "f64", "f32"]])
@pytest.mark.parametrize("n,nu2", [(15, 2), (31, 3), (63, 2), (127, 2)])
def test_prolong_two_sweeps_bitwise(n, nu2, fmt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"prolong + 2 sweeps n={n} nu2={nu2} {fmt}", flush=True)
    m = mgir.full_levels(n)
    prec = [fmt[min(i, len(fmt) - 1)] for i in range(m)]
    g = torch.Generator(device="cuda").manual_seed(n)
    b = (torch.rand((n,) * 3, dtype=torch.float64, device="cuda", generator=g) - 0.5).to(mgir.TORCH_DTYPE[prec[0]])
    got, want = (mgir.Solver(3, n, prec, nu2=nu2) for _ in range(2))
    for s in (got, want):
        s.set_shape(0, mgir.SHAPE_TAIL, [0])  # every level by launches of its own
    for l in range(m - 1):
        sh = want.get_shape(l, mgir.SHAPE_SWEEP)
        want.set_shape(l, mgir.SHAPE_SWEEP, sh)
    c = want.vcycle(b).clone()
    for _ in range(2):
        assert torch.equal(got.vcycle(b), c)
