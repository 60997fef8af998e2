"""The fused tile kernels of the 2-D levels: the cycle against the stage kernels
(bitwise), and the finest level's update against its definition, on grids with
whole and ragged tiles, both discretisations, one to three sweeps."""
import numpy as np
import pytest
import torch

import oracle
from paper_2007_07539_amd import mgir
from paper_2007_07539_amd import workloads as W
from tests.helpers import round_to

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,disc,fmt,nu1,nu2", [
    (127, "fd", ["f64"], 1, 3), (255, "fd", ["f16", "f32", "f64"], 2, 2), (511, "fd", ["bf16"], 3, 1),
    (1023, "fd", ["f32", "f64"], 2, 2), (131, "q1", ["f16"], 2, 2), (191, "q1", ["f64", "f16"], 3, 3),
    (575, "q1", ["f16"] * 3 + ["f64"], 2, 1), (4095, "q1", ["f16"], 2, 2)])
def test_tile_cycle_equals_the_stages(n, disc, fmt, nu1, nu2):
    m = mgir.full_levels(n)
    prec = [fmt[min(i, len(fmt) - 1)] for i in range(m)]
    print(f"2-D tiles n={n} {disc} {prec[:3]} V({nu1},{nu2})", flush=True)
    s = mgir.Solver(2, n, prec, nu1=nu1, nu2=nu2, disc=disc)
    b = torch.from_numpy(W.uniform_rhs(2, n, seed=4)).to("cuda").to(mgir.TORCH_DTYPE[prec[0]])
    c = s.vcycle(b).double()
    b1 = s.read(1, mgir.BUF_RHS)
    for l in range(m - 1):
        s.stage(mgir.STAGE_SMOOTH_FIRST, l)
        s.stage(mgir.STAGE_RESTRICT, l)
    s.stage(mgir.STAGE_COARSE, m - 1)
    for l in range(m - 2, -1, -1):
        s.stage(mgir.STAGE_PROLONG_SWEEP, l)
        for _ in range(nu2 - 1):
            s.stage(mgir.STAGE_SWEEP, l)
    assert c.abs().max() > 0
    assert torch.equal(b1, s.read(1, mgir.BUF_RHS))
    assert torch.equal(c, s.read(0, mgir.BUF_COR))


@pytest.mark.parametrize("n,disc,name,defer", [
    (127, "fd", "f16", 0), (255, "fd", "f64", 0), (511, "fd", "hsd", 0), (131, "q1", "f16", 2), (191, "q1", "f64", 0),
    (575, "q1", "f32", 3)])
def test_tile_update_is_the_step(n, disc, name, defer):
    """One refinement step from u = 0: u = alpha f c with c the V-cycle of the
    scaled right-hand side (bitwise), and the norm of r = b - A u, formed in
    FP64 (1e-12: two orders of summation)."""
    print(f"2-D fused update n={n} {disc} {name} defer={defer}", flush=True)
    prec = W.precision_map(name, mgir.full_levels(n))
    b = W.uniform_rhs(2, n, seed=5)
    bt = torch.from_numpy(b).to("cuda")
    s = mgir.Solver(2, n, prec, disc=disc, defer_update=defer, residual_scaling=name != "f64", max_iter=1)
    u, res = s.solve(bt, check=False)
    assert res.iterations == 1
    alpha = 2.0 ** s.alpha_shift() * float(np.abs(b).max()) if name != "f64" else 1.0
    v = mgir.Solver(2, n, prec, disc=disc)
    # (a single correct rounding; torch's double-to-half conversion rounds twice)
    bh = torch.from_numpy(round_to(b * (1.0 / alpha), prec[0])).to("cuda").to(mgir.TORCH_DTYPE[prec[0]])
    c = v.vcycle(bh).double()
    f = 1.0 if disc == "q1" else (1.0 / (n + 1)) * (1.0 / (n + 1))
    assert torch.equal(u, (alpha * f) * c)
    r = oracle.residual(b, u.cpu().numpy(), disc)
    assert abs(res.history[1] / (oracle.norm2(r) / oracle.norm2(b)) - 1.0) <= 1e-12


@pytest.mark.parametrize("n,name,scaling", [(127, "f16", True), (255, "f64", False), (511, "f32", True),
                                            (2047, "f16", True)])
def test_autotuned_tiles_have_the_same_history(n, name, scaling, tmp_path, monkeypatch):
    """An autotuned 2-D handle sums the norm partials of every tile: u and the
    iterations are the untuned handle's, freshly timed and read from the tuning
    cache, and so are the norms, up to their summation order (n^2 eps at most, far
    below 1e-8)."""
    print(f"autotuned 2-D tiles n={n} {name}", flush=True)
    monkeypatch.setenv("MGIR_TUNE_CACHE", str(tmp_path / "tune.txt"))
    prec = W.precision_map(name, mgir.full_levels(n))
    b = torch.from_numpy(W.uniform_rhs(2, n, seed=6)).to("cuda")
    u0, r0 = mgir.Solver(2, n, prec, residual_scaling=scaling).solve(b)
    for fresh in (True, False):
        u, r = mgir.Solver(2, n, prec, residual_scaling=scaling, autotune=True).solve(b)
        assert r.iterations == r0.iterations and torch.equal(u, u0), fresh
        assert np.allclose(r.history, r0.history, rtol=1e-8, atol=0.0), (fresh, r.history, r0.history)
