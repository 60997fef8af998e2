"""GPU: the marching Q1 sweep and residual (FP32, FP64) with each number of
planes per thread that its rule gives (2, 4, 8, 16), last chunks ragged, against
the oracle with the tolerances of the other Q1 stage tests."""
import pytest

from tests import test_gpu_q1 as q1

pytestmark = pytest.mark.gpu
dev = q1.dev


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [27, 55, 79, 111, 135])
def test_q1_march_planes(dev, ref, prec, n):
    q1.test_q1_sweep(dev, ref, prec, 3, n)
    q1.test_q1_resid_restrict(dev, ref, prec, prec, 3, n)
