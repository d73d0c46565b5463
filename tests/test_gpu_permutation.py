"""Row interchanges of partial pivoting applied as one permutation, around the
orders where it moves from LDS (up to 16384, of which more than 12288 need above
64 KB) to global memory, and a pivoted solve above them."""
import numpy as np
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


@pytest.mark.parametrize("n", [1, 33, 511, 12289, 16383, 16384, 16385])
def test_interchanges_in_order(rbt, n):
    """Random valid interchanges and identity factors: B's rows, exactly."""
    rng = np.random.default_rng(n)
    ipiv = rng.integers(np.arange(n), n) + 1
    ipiv[::7] = np.arange(n)[::7] + 1  # some of them none
    want = np.arange(n)
    for j, p in enumerate(ipiv - 1):
        want[[j, p]] = want[[p, j]]
    LU = torch.eye(n, dtype=torch.float64, device="cuda").t()
    B = torch.arange(2 * n, dtype=torch.float64, device="cuda").reshape(2, n).t()
    X = rbt.gepp_solve(LU, torch.from_numpy(ipiv).cuda(), B.clone())
    assert torch.equal(X, B[torch.from_numpy(want).cuda()])


def test_pivoted_solve_above_the_lds_order(rbt):
    n = 16500
    A = workloads.device_randn(n, n, 5)
    B = workloads.device_randn(n, 2, 6)
    LU, ipiv, info = rbt.gepp(A.clone())
    assert int(info) == 0
    X = rbt.gepp_solve(LU, ipiv, B.clone())
    R = (B - A @ X).abs().amax(0)
    bound = 10 * n * EPS * (A.abs().sum(1).max() * X.abs().amax(0) + B.abs().amax(0))
    assert bool((R <= bound).all())
