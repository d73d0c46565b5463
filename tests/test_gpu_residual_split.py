"""The residual's two forms for many right-hand sides, on either side of the
number of 64 x 64 tiles where it changes from one to the other (one and a half
per compute unit with partial tiles, one without), against torch in FP64."""
import pytest
import torch

from paper_2312_09376_amd import workloads

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def rbt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_09376_amd import rbt as r
    r.lib()
    return r


@pytest.mark.parametrize("n,k", [(1500, 900), (1500, 961), (1001, 1600), (1024, 960), (1024, 1024)])
def test_backward_error_of_many_right_hand_sides(rbt, n, k):
    """Sums of n + 1 terms, each at most the denominator's: 2 (n + 2) eps."""
    A = workloads.device_randn(n, n, 1)
    X, B = workloads.device_randn(n, k, 2), workloads.device_randn(n, k, 3)
    R = B - A @ X
    an = A.abs().sum(1).max()
    ref = (R.abs().amax(0) / (an * X.abs().amax(0) + B.abs().amax(0))).max()
    assert abs(float(rbt.backward_error(A, X, B)) - float(ref)) <= 2 * (n + 2) * EPS
