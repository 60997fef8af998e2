"""GPU: large grids postpone their solution updates by default (a ring of eight
corrections); u is bit for bit that of updating in place, over a full ring and a
remainder, from zero and from a guess, on repeated solves."""
import ctypes

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


def _rebind(s, nbytes):
    """Bind another workspace of nbytes, every byte of it 0xff (a NaN in every format) before."""
    s.workspace = torch.full((nbytes + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    base = s.workspace.data_ptr()
    st = mgir._stream_ptr(None)
    return s.lib.mg_bind_workspace(s._h, ctypes.c_void_p(base + (-base) % 256), nbytes, st)


def _b(shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(shape, dtype=torch.float64, device="cuda", generator=g) - 0.5


@pytest.mark.parametrize("dim,n,name,disc", [(3, 255, "f16", "fd"), (2, 2303, "f16", "q1"), (2, 255, "f64", "fd")])
def test_optional_parts_of_the_workspace(dim, n, name, disc):
    """A workspace without room for the default ring (or the second residual of a
    2-D FP64 grid) is taken, on its own and after a full one, and gives the same
    u; one byte less is refused.  defer_update = -1 asks for that size, and runs
    no postponed update."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"optional workspace {dim}-D n={n} {name} {disc}", flush=True)
    prec = W.precision_map(name, mgir.full_levels(n))
    kw = dict(disc=disc, residual_scaling=name != "f64", max_iter=9, rtol=0.0)
    b = _b((n,) * dim, n) / (float(n + 1) ** dim if disc == "q1" else 1.0)
    s = mgir.Solver(dim, n, prec, **kw)
    never = mgir.Solver(dim, n, prec, defer_update=-1, **kw)
    small = never.workspace_bytes
    if name == "f64":
        small -= ((n + 3) * (n + 1) * 8 + 255) // 256 * 256
    else:
        assert small < s.workspace_bytes
        assert not any("defer" in r[0] for r in never.profile_step())
    u = s.solve(b, check=False)[0].clone()
    assert torch.equal(never.solve(b, check=False)[0], u)
    full = s.workspace_bytes
    assert _rebind(s, small - 1) == mgir.MG_ERR_WORKSPACE
    for nbytes in (small, full, small):
        assert _rebind(s, nbytes) == mgir.MG_OK
        for _ in range(2):
            assert torch.equal(s.solve(b, check=False)[0], u), nbytes


@pytest.mark.parametrize("dim,n,name,disc", [(3, 31, "f16", "fd"), (3, 31, "f32", "fd"), (3, 9, "f16", "q1"),
                                             (3, 31, "f16", "q1"), (3, 13, "f64", "q1"), (2, 13, "bf16", "q1"),
                                             (2, 131, "f16", "q1")])
def test_ring_in_a_workspace_of_nans(dim, n, name, disc):
    """Binding clears the rings too: u is that of updates in every step, whatever the
    workspace held before."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"ring in a dirty workspace {dim}-D n={n} {name} {disc}", flush=True)
    prec = W.precision_map(name, mgir.full_levels(n))
    kw = dict(disc=disc, residual_scaling=name != "f64", max_iter=7, rtol=0.0)
    b = _b((n,) * dim, n) / (float(n + 1) ** dim if disc == "q1" else 1.0)
    u = mgir.Solver(dim, n, prec, defer_update=-1, **kw).solve(b, check=False)[0]
    s = mgir.Solver(dim, n, prec, defer_update=3, **kw)
    assert _rebind(s, s.workspace_bytes) == mgir.MG_OK
    for _ in range(2):
        assert torch.equal(s.solve(b, check=False)[0], u)


@pytest.mark.parametrize("cols", [False, True])
def test_group_workspace_without_rings(cols):
    """A batch and a handle of columns take a workspace without room for their rings."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"group workspace cols={cols}", flush=True)
    prec = W.precision_map("f16", mgir.full_levels(31))
    make = (lambda: mgir.MultiSolver(31, 8, prec)) if cols else (lambda: mgir.BatchedSolver([31, 7, 31], prec))
    b = _b((31, 31, 31, 8), 3) if cols else [_b((n,) * 3, n) for n in (31, 7, 31)]
    s = make()
    u = s.solve(b)[0]
    ring = 8 * 33 * 32 * 32 * 2 * (8 if cols else 2)  # (plus smaller parts)
    for nbytes in (s.workspace_bytes - ring, s.workspace_bytes):
        assert _rebind(s, nbytes) == mgir.MG_OK
        v = s.solve(b)[0]
        assert torch.equal(u, v) if cols else all(torch.equal(x, y) for x, y in zip(u, v))
