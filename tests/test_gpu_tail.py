"""The fused coarse end (one workgroup, levels in LDS) against the level kernels
it replaces, run stage by stage on the same handle: bitwise the same vectors on
every level, in 2-D and 3-D, both discretisations, with a one-point base and
with a CG base, where the whole cycle fits the kernel and where only its end does."""
import pytest
import torch

from paper_2007_07539_amd import mgir
from paper_2007_07539_amd import workloads as W

pytestmark = pytest.mark.gpu

CASES = [
    # dim, n, disc, nlevels, formats (the last one repeats), nu1, nu2
    (3, 3, "fd", 0, ["f16", "f64"], 2, 2), (3, 15, "fd", 0, ["f64"], 2, 2), (3, 31, "fd", 0, ["f16"], 1, 1),
    (3, 15, "fd", 0, ["bf16"] * 3 + ["f32"], 3, 2), (3, 31, "fd", 3, ["f16"] * 2 + ["f64"], 2, 1),
    (2, 3, "fd", 0, ["f64"], 2, 2), (2, 63, "fd", 0, ["f32", "f16", "bf16", "f16", "f32", "f64"], 2, 3),
    (2, 127, "fd", 0, ["f64"] * 6 + ["f16"], 2, 2), (2, 63, "fd", 3, ["f16"], 4, 2),
    (3, 7, "q1", 0, ["f16"], 2, 2), (3, 15, "q1", 0, ["f64"], 1, 2), (3, 11, "q1", 0, ["f32", "f64"], 2, 2),
    (3, 13, "q1", 0, ["f16"], 2, 1), (3, 9, "q1", 0, ["bf16"], 3, 3), (3, 47, "q1", 0, ["f16"] * 4 + ["f64"], 2, 2),
    (2, 63, "q1", 0, ["f16"], 2, 2), (2, 23, "q1", 0, ["f64"], 2, 2), (2, 95, "q1", 0, ["bf16"] * 5 + ["f64"], 3, 1),
]


@pytest.mark.parametrize("dim,n,disc,nlevels,fmt,nu1,nu2", CASES)
def test_fused_coarse_end_equals_the_stages(dim, n, disc, nlevels, fmt, nu1, nu2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = nlevels or mgir.full_levels(n)
    prec = [fmt[min(i, len(fmt) - 1)] for i in range(m)]
    print(f"fused coarse end {dim}-D n={n} {disc} {prec} V({nu1},{nu2})", flush=True)
    s = mgir.Solver(dim, n, prec, nu1=nu1, nu2=nu2, disc=disc, nlevels=nlevels)
    b = torch.from_numpy(W.uniform_rhs(dim, n, seed=3)).to("cuda").to(mgir.TORCH_DTYPE[prec[0]])
    c = s.vcycle(b).double()
    fused = [(s.read(l, mgir.BUF_RHS), s.read(l, mgir.BUF_COR)) for l in range(1, m)]
    # the same cycle, one launch per stage
    for l in range(m - 1):
        s.stage(mgir.STAGE_SMOOTH_FIRST, l)
        s.stage(mgir.STAGE_RESTRICT, l)
    s.stage(mgir.STAGE_COARSE, m - 1)
    for l in range(m - 2, -1, -1):
        s.stage(mgir.STAGE_PROLONG_SWEEP, l)
        for _ in range(nu2 - 1):
            s.stage(mgir.STAGE_SWEEP, l)
    assert c.abs().max() > 0
    assert torch.equal(c, s.read(0, mgir.BUF_COR))
    for l in range(1, m):
        assert torch.equal(fused[l - 1][0], s.read(l, mgir.BUF_RHS)), ("right-hand side of level", l)
        assert torch.equal(fused[l - 1][1], s.read(l, mgir.BUF_COR)), ("correction of level", l)
