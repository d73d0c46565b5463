"""The slab kernel of the partial-pivoting elimination at the sizes where its
split changes: one workgroup and several (512 rows each), slabs narrower than
32 columns, one and two rows per thread (more than 16384 rows is the second),
and the column-by-column path that a small workspace selects. Pivots are
compared with the oracle's (N(0,1) entries: no ties) and factors within the
componentwise bound of two orderings of the same elimination."""
import numpy as np
import pytest
import torch

from oracle import pivoted
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.T)).cuda().t()


def host(t):
    return t.detach().cpu().numpy()


def check(rbt, A, work=None):
    n = A.shape[0]
    LU, ipiv, info = rbt.gepp(dev(A), work=work)
    LUo, ipiv_o, info_o = pivoted.gepp(A)
    assert int(info.item()) == info_o
    assert np.array_equal(host(ipiv), ipiv_o)
    den = np.abs(np.tril(LUo, -1) + np.eye(n)) @ np.abs(np.triu(LUo))
    assert (np.abs(host(LU) - LUo) <= 4 * n * EPS * den + 1e-300).all()


@pytest.mark.parametrize("n", [31, 32, 33, 64, 511, 512, 513, 640, 1025])
def test_slab_edges_match_oracle(rbt, n):
    check(rbt, workloads.randn_matrix(n, seed=n + 7))


def test_small_workspace_takes_columns(rbt):
    n = 700
    work = torch.empty(8192, dtype=torch.uint8, device="cuda")
    check(rbt, workloads.randn_matrix(n, seed=3), work=work)


def test_ties_take_the_first_row(rbt):
    """Entries +-1: every column of the first slab has many rows of the largest
    magnitude, in several workgroups; the first one is the pivot (LAPACK's
    idamax), also among rows swapped in earlier."""
    n = 1100
    A = np.sign(workloads.randn_matrix(n, seed=11))
    A[:, 1:] += 0.25 * workloads.randn_matrix(n, seed=12)[:, 1:]
    check(rbt, A)


def test_two_rows_per_thread(rbt):
    """More than 16384 rows: two rows per thread. P A = L U on sampled rows."""
    n = 16500
    A = workloads.device_randn(n, n, 5)
    LU, ipiv, info = rbt.gepp(A.clone())  # (clone keeps the column-major strides)
    assert int(info.item()) == 0
    perm = np.arange(n)
    for j, p in enumerate(host(ipiv) - 1):
        perm[[j, p]] = perm[[p, j]]
    assert np.array_equal(np.sort(perm), np.arange(n))
    rows = np.array([0, 1, 31, 32, 127, 128, 5000, 16383, 16384, n - 1])
    L = torch.tril(LU, -1)
    U = torch.triu(LU)
    Ls = L[rows].clone()
    Ls[np.arange(len(rows)), rows] = 1.0
    got = Ls @ U
    want = A[torch.from_numpy(perm[rows]).cuda()]
    bound = n * EPS * (Ls.abs() @ U.abs())
    assert bool(((got - want).abs() <= bound).all())
    assert float(L.abs().max()) <= 1.0


def test_expired_exchange_leaves_no_finite_factors(rbt):
    """A wait that expires (forced from the host: every wait expires at once,
    every kernel still exits) is never a silently wrong factorization."""
    from paper_2312_09376_amd import _lib
    A = dev(workloads.randn_matrix(1200, seed=4))
    old = rbt.get_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT)
    rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, -1)
    try:
        LU, _, _ = rbt.gepp(A)
        torch.cuda.synchronize()
    finally:
        rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, old)
    assert bool(torch.isnan(LU).any())
