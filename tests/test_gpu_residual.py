"""The residual and its backward error around the edges of the product's
tiles (16 rows, runs of 32 columns, eight wavefronts, 16 / 32 / 64 right-hand
sides and the GEMM beyond), leading dimensions above n, both transposes."""
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


def dev(a, pad=0):
    n, k = a.shape
    t = torch.full((k, n + pad), float("nan"), dtype=torch.float64, device="cuda")
    t[:, :n] = torch.from_numpy(np.ascontiguousarray(a.T)).cuda()
    return t.t()[:n]


@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 33, 64, 65])
@pytest.mark.parametrize("n", [1, 2, 15, 17, 31, 33, 255, 257, 300])
def test_backward_error(rbt, n, k):
    """|error| <= 2 (n + 2) eps: each residual entry is a sum of n + 1 terms
    of at most ||A|| max|X| and max|B|, the denominator's terms."""
    A = workloads.randn_matrix(n, seed=n)
    X, B = workloads.randn(n, k, seed=k), workloads.randn(n, k, seed=k + 1)
    R = B - A @ X
    an = np.abs(A).sum(axis=1).max()
    ref = (np.abs(R).max(0) / (an * np.abs(X).max(0) + np.abs(B).max(0))).max()
    be = float(rbt.backward_error(dev(A, 3), dev(X, 1), dev(B, 2)))
    assert abs(be - ref) <= 2 * (n + 2) * EPS


@pytest.mark.parametrize("n,k", [(4097, 3), (4100, 16), (1024, 1024), (1000, 1030)])
def test_backward_error_larger(rbt, n, k):
    A = workloads.device_randn(n, n, 1)
    X, B = workloads.device_randn(n, k, 2), workloads.device_randn(n, k, 3)
    R = B - A @ X
    an = A.abs().sum(1).max()
    ref = (R.abs().amax(0) / (an * X.abs().amax(0) + B.abs().amax(0))).max()
    assert abs(float(rbt.backward_error(A, X, B)) - float(ref)) <= 2 * (n + 2) * EPS


def test_nan_never_looks_converged(rbt):
    n, k = 300, 5
    A, X, B = workloads.dominant(n, seed=1), np.zeros((n, k)), np.ones((n, k))
    for where in [(0, 0), (299, 4), (130, 2)]:
        Bn = B.copy()
        Bn[where] = np.nan
        assert np.isnan(float(rbt.backward_error(dev(A), dev(X), dev(Bn))))


@pytest.mark.parametrize("n,k", [(1, 1), (17, 2), (130, 16), (257, 17), (300, 64), (515, 5)])
def test_adjoint(rbt, n, k):
    A = workloads.dominant(n, seed=n + 1)
    B, G = workloads.randn(n, k, seed=5), workloads.randn(n, k, seed=6)
    X, LU, _, _, _, _ = rbt.solve_mixed(dev(A), dev(B), 2, 2023, prec=rbt.RBT_FP32,
                                        solver=rbt.RBT_IR_CLASSIC)
    _, dB, _, berr = rbt.solve_backward_mixed(LU, dev(A), X, dev(G), 2, 2023)
    ref = np.linalg.solve(A.T, G)
    assert float(berr.item()) <= 10 * n * EPS
    assert np.linalg.norm(dB.cpu().numpy() - ref) <= 100 * n * EPS * np.linalg.norm(ref)
