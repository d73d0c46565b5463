"""The triangular sweeps in every form the dispatch can choose: one
right-hand side, groups of 4, 8 and 16 (by order and number of right-hand
sides), several groups side by side, the last of them ragged, the block solves beyond 384, both transposes, orders
around one and two blocks, a leading dimension above n, and a workspace with
no room for more than one group. FP64 factors: against the oracle's
triangular solves. FP32 factors: the refined solution and adjoint."""
import numpy as np
import pytest
import torch

from oracle import solve as osolve
from paper_2312_09376_amd import _lib, workloads

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


def host(t):
    return t.detach().cpu().numpy()


def relfro(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def expected(LUo, B, trans):
    if trans == 0:
        return osolve.lu_solve(LUo, B)
    return osolve.backward_unit_lower_transposed(LUo, osolve.forward_upper_transposed(LUo, B))


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("n,k", [(1, 2), (7, 5), (127, 1), (128, 4), (129, 8), (255, 9), (256, 16),
                                 (257, 17), (300, 1), (385, 33), (130, 384), (130, 385)])
def test_getrs_forms(rbt, n, k, trans):
    A = workloads.dominant(n, seed=n + 1)
    B = workloads.randn(n, k, seed=9)
    LUo, _ = osolve.genp_unblocked(A)
    X = rbt.getrs(dev(LUo, pad=3), dev(B, pad=1), trans=trans)
    assert relfro(host(X), expected(LUo, B, trans)) <= 1e-12


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("n,k", [(2049, 383), (4200, 375)])
def test_wide_groups(rbt, n, k, trans):
    """Groups of 8 and of 16: the residual within the bound of two triangular
    solves, 2 n eps |L| |U| |X| (the product for the residual adds as much)."""
    A = workloads.device_shifted(n, 1)
    LU, _ = rbt.genp(A)
    B = workloads.device_randn(n, k, 2)
    X = rbt.getrs(LU, B.clone(), trans=trans)
    L = torch.tril(LU, -1) + torch.eye(n, dtype=LU.dtype, device="cuda")
    U = torch.triu(LU)
    if trans:
        L, U = U.t().contiguous(), L.t().contiguous()
    R = (B - L @ (U @ X)).abs()
    bound = 4 * n * EPS * (L.abs() @ (U.abs() @ X.abs()))
    assert bool((R <= bound).all())


@pytest.mark.parametrize("k", [16, 40])
def test_getrs_workspace_without_publication_buffer(rbt, k):
    """A workspace that ends with the sweeps' area (smaller than
    rbt_workspace_size for 40 right-hand sides) is still accepted."""
    n = 300
    A = workloads.dominant(n, seed=5)
    B = workloads.randn(n, k, seed=2)
    LUo, _ = osolve.genp_unblocked(A)
    nb = (n + 127) // 128
    sync = ((64 + 2 * 16 * n) * 4 + 255) // 256 * 256
    work = torch.empty(nb * 2 * 128 * 128 * 8 + sync, dtype=torch.uint8, device="cuda")
    X = rbt.getrs(dev(LUo), dev(B), trans=0, work=work)
    assert relfro(host(X), expected(LUo, B, 0)) <= 1e-12


@pytest.mark.parametrize("n,k", [(129, 1), (257, 3), (300, 16), (515, 17), (260, 40), (1100, 383)])
def test_mixed_forms(rbt, n, k):
    A = workloads.dominant(n, seed=n)
    B = workloads.randn(n, k, seed=4)
    G = workloads.randn(n, k, seed=6)
    X, LU, _, berr, _, _ = rbt.solve_mixed(dev(A), dev(B), 2, 2023, prec=rbt.RBT_FP32,
                                           solver=rbt.RBT_IR_CLASSIC)
    assert float(berr.item()) <= 10 * n * EPS
    assert relfro(host(X), np.linalg.solve(A, B)) <= 100 * n * EPS
    _, dB, _, berr = rbt.solve_backward_mixed(LU, dev(A), X, dev(G), 2, 2023)
    assert float(berr.item()) <= 10 * n * EPS
    assert relfro(host(dB), np.linalg.solve(A.T, G)) <= 100 * n * EPS


def test_groups_expired_wait_is_nan(rbt):
    n, k = 400, 40
    A = workloads.dominant(n, seed=3)
    LU, _ = rbt.genp(dev(A))
    default = rbt.get_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT)
    try:
        rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, -1)
        X = host(rbt.getrs(LU, dev(workloads.randn(n, k, seed=9)), trans=0))
    finally:
        rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, default)
    assert not np.isfinite(X[256:]).any()  # (the last block row waits in both sweeps)
