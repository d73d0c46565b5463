"""Triangular solves and factors beside an exact zero pivot: what is solved or
factored before it must stay what plain substitution gives, whichever path
(sweeps with inverses, block solves, block kernels) the number of right-hand
sides and the workspace select."""
import numpy as np
import pytest
import torch

from paper_2312_09376_amd import workloads
from tests.ieee import same_nonfinite, substitution, tame

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rbt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_09376_amd import rbt as r
    r.lib()
    return r


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.T)).cuda().t()


def host(t):
    return t.detach().cpu().numpy()


def tri(n, seed):
    """L\\U whose triangles are well conditioned at any order."""
    F = workloads.randn_matrix(n, seed=seed) / n
    F[np.arange(n), np.arange(n)] = 1.0 + 0.1 * np.arange(n) / n
    return F


@pytest.mark.parametrize("full", [True, False])
@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("n,k,at", [(300, 17, 200), (300, 40, 127), (257, 100, 256), (200, 384, 0),
                                    (1200, 300, 1030)])
def test_solve_beside_a_zero_on_the_diagonal(rbt, n, k, at, trans, full):
    """17 to 384 right-hand sides, with the whole workspace (sweeps) and with one
    that ends after the sweeps' area (block solves)."""
    LU = tri(n, seed=n)
    LU[at, at] = 0.0
    B = workloads.randn(n, k, seed=3)
    L, U = np.tril(LU, -1) + np.eye(n), np.triu(LU)
    if trans == 0:
        want = substitution(U, substitution(L, B, True, True), False, False)
    else:
        want = substitution(L.T, substitution(U.T, B, True, False), False, True)
    work = None
    if not full:
        nb = (n + 127) // 128
        sync = ((64 + 2 * 16 * n) * 4 + 255) // 256 * 256
        work = torch.empty(nb * 2 * 128 * 128 * 8 + sync, dtype=torch.uint8, device="cuda")
    X = rbt.getrs(dev(LU), dev(B), trans=trans, work=work)
    same_nonfinite(host(X), want)


def test_solve_with_one_infinite_right_hand_side(rbt):
    n, k = 300, 64
    LU = tri(n, seed=1)
    B = workloads.randn(n, k, seed=3)
    B[140, 5] = np.inf
    L, U = np.tril(LU, -1) + np.eye(n), np.triu(LU)
    y = substitution(L, B, True, True)
    X = rbt.getrs(dev(LU), dev(B), trans=0)
    same_nonfinite(host(X), substitution(U, y, False, False))


@pytest.mark.parametrize("at", [3, 40, 150, 290])
def test_factors_beside_a_zero_pivot(rbt, at):
    """A leading block that becomes singular: L's columns before it and U's rows
    up to it right of its 16-column step are those of plain elimination."""
    n = 300
    A = tame(n, np.float64)
    F = A.copy()
    for j in range(at):
        F[j + 1:, j] /= F[j, j]
        F[j + 1:, j + 1:] -= np.outer(F[j + 1:, j], F[j, j + 1:])
    A[at, :at + 1] = 0.0
    F[at, :at] = 0.0
    F[at, at:] = A[at, at:]
    LU, info = rbt.genp(dev(A))
    assert int(info) == at + 1
    got, right = host(LU), 16 * (at // 16 + 1)
    same_nonfinite(got[:at + 1, right:], F[:at + 1, right:])
    same_nonfinite(got[:, :at], F[:, :at])


@pytest.mark.parametrize("n,at", [(200, 70), (700, 133)])
def test_pivoted_factors_beside_a_zero_column(rbt, n, at):
    """Partial pivoting of a matrix with a zero column: U's rows above it."""
    A = workloads.randn_matrix(n, seed=n)
    A[:, at] = 0.0
    LU, ipiv, info = rbt.gepp(dev(A))
    assert int(info) == at + 1
    U = np.triu(host(LU))[:at]
    assert np.isfinite(U).all()
    perm = np.arange(n)
    for j, p in enumerate(host(ipiv)[:at] - 1):
        perm[[j, p]] = perm[[p, j]]
    L = np.tril(host(LU)[:at, :at], -1) + np.eye(at)
    err = np.abs(L @ U - A[perm[:at]])
    assert (err <= 4 * n * 2.0 ** -52 * (np.abs(L) @ np.abs(U))).all()
