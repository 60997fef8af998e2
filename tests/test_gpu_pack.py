"""GPU: dense <-> padded copies (written and read levels, V-cycle input and
output) around the eight-point, four-point and two-point rows of the copy
kernel: rows shorter than one access, of exactly one, and with an overlapping
last access; every pair of formats, in 2-D and 3-D.  The copies convert with one
rounding, so the expected values are exact."""
import numpy as np
import pytest
import torch

from paper_2007_07539_amd import mgir
from tests.helpers import round_to

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("dim,n", [(3, 3), (3, 7), (3, 9), (3, 15), (3, 23), (2, 7), (2, 9), (2, 31), (2, 47)])
def test_pack_unpack_exact(dim, n, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"pack {dim}-D n={n} {prec}", flush=True)
    s = mgir.Solver(dim, n, [prec] * mgir.full_levels(n), disc="q1" if (n + 1) & n else "fd")
    x = np.random.default_rng(n).uniform(-100, 100, (n,) * dim)
    names = {torch.float64: "f64", torch.float32: "f32", torch.float16: "f16", torch.bfloat16: "bf16"}
    for src, name in names.items():
        xs = round_to(x, name)  # a value of the source format, then one rounding to the level's
        t = torch.from_numpy(xs).to("cuda").to(src)
        s.write(0, mgir.BUF_RHS, t)
        want = round_to(xs, prec)
        assert np.array_equal(s.read(0, mgir.BUF_RHS, dtype=torch.float64).cpu().numpy(), want), name
        for dst, dname in names.items():
            got = s.read(0, mgir.BUF_RHS, dtype=dst).double().cpu().numpy()
            assert np.array_equal(got, round_to(want, dname)), (name, dname)
