"""Tensor blocks whose Gram matrices are formed in ranges, against the oracle (bars of test_gpu_parity.py)."""
import pytest

from paper_2309_06497_amd import workloads as wl
from test_gpu_parity import TensorPair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("last,bf16", [(2, False), (9, True), (15, False), (16, False), (17, False)])
def test_last_dimension_around_the_narrow_gram_kernel(last, bf16):
    """Row counts that 16 does not divide, columns up to and just above one 16-wide tile; the first and
    the middle unfolding (k = 24 * last ...) are cut into one range, several, and a short last one."""
    shapes = [(20, 24, last), (7, 23, last), (9,)]
    p = TensorPair(shapes, 24, 0.99, 2, bf16=bf16)
    for t in range(3):
        p.step(wl.gaussian_grads(shapes, 71, t, 1e-2), 0.01, t)
        p.check(t)


def test_more_tensors_than_one_copy_launch_holds():
    shapes = [(3, 5, 7), (4, 6, 2), (5, 5, 5)] * 9 + [(6, 7)]
    p = TensorPair(shapes, 6, 0.99, 1)
    for t in range(2):
        p.step(wl.gaussian_grads(shapes, 72, t, 1e-2), 0.01, t)
        p.check(t)
