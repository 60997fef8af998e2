"""GPU: the LDS-plane march at the edges of its tiles: one, two, three and all
rows per block and planes per chunk (chunks starting on even and odd planes,
rows past the grid, the last coarse row), for the sweeps, the prolongation and
the restriction, in each format and with mixed fine and coarse formats.  A launch
shape only cuts the work differently, so every V-cycle equals the one of the
register-queue kernels (ty = 0) bit for bit."""
import pytest
import torch

from paper_2007_07539_amd import mgir

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fine,coarse", [("f16", "f16"), ("f16", "f32"), ("bf16", "f16"), ("f32", "bf16"), ("f64", "f64"),
                                         ("f32", "f64")])
@pytest.mark.parametrize("n", [15, 31])
def test_march_shapes_bitwise(n, fine, coarse):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"march n={n} {fine}/{coarse}", flush=True)
    m = mgir.full_levels(n)
    s = mgir.Solver(3, n, [fine] + [coarse] * (m - 1), nu1=3, nu2=2)
    g = torch.Generator(device="cuda").manual_seed(n)
    b = (torch.rand((n,) * 3, dtype=torch.float64, device="cuda", generator=g) - 0.5).to(mgir.TORCH_DTYPE[fine])
    s.set_shape(0, mgir.SHAPE_TAIL, [0])
    kinds = (mgir.SHAPE_SMOOTH, mgir.SHAPE_SWEEP, mgir.SHAPE_PROLONG)
    for k in kinds:
        s.set_shape(0, k, [4, n, 256, 1, 0])
    want = s.vcycle(b).clone()
    tried = 0
    for V in (4, 8):
        for ty in (1, 2, 3, n):
            for zc in (1, 2, 3, n):
                for dp, sg in ((1, 0), (2, 0), (1, 1)):
                    try:
                        for k in kinds:
                            s.set_shape(0, k, [V, zc, 256, 1, ty, dp, sg if k == mgir.SHAPE_PROLONG else 1])
                    except mgir.MgError:
                        continue
                    assert torch.equal(s.vcycle(b), want), (V, ty, zc, dp, sg)
                    tried += 1
    assert tried >= 40
    for V in (4, 8):
        for tyc, zcc, pipe in ((1, 1, 1), (2, 3, 1), (n // 2, n // 2, 1), (3, 2, 2)):
            try:
                s.set_shape(0, mgir.SHAPE_RESTRICT, [V, tyc, zcc, pipe])
            except mgir.MgError:
                continue
            assert torch.equal(s.vcycle(b), want), (V, tyc, zcc, pipe)
