"""Batches whose large systems are solved by teams of 2, 4 and 8 workgroups
(few systems of order 512 and more): solutions against LAPACK, the FP64
fallback, a zero pivot in a strip of a later member, and identical results
on every launch (the members' meeting order varies)."""
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a.T)).cuda().t()


def host(t):
    return t.detach().cpu().numpy()


def relfro(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("ns,ks,depth", [([512], [1], 2), ([513, 511, 40], [3, 2, 1], 2),
                                         ([1024, 1023, 600], [16, 1, 5], 1),
                                         ([1500, 900, 700, 64, 130], [4, 2, 9, 1, 1], 4)])
def test_teams_match_lapack(rbt, prec, ns, ks, depth):
    p = rbt.RBT_FP32 if prec == "fp32" else rbt.RBT_BF16
    As = [workloads.dominant(n, seed=n) for n in ns]
    Bs = [workloads.randn(n, k, seed=n + 1) for n, k in zip(ns, ks)]
    plan = rbt.batched_plan(ns, ks, depth=depth, prec=p)
    Ad, Bd = [dev(a) for a in As], [dev(b) for b in Bs]
    Xs, iters, berr, info = rbt.solve_batched(plan, Ad, Bd, seed=7)
    first = [x.clone() for x in Xs]
    for s, (n, A, B) in enumerate(zip(ns, As, Bs)):
        assert int(info[s]) == 0 and float(berr[s]) <= 10 * n * EPS, (n, float(berr[s]))
        assert relfro(host(Xs[s]), np.linalg.solve(A, B)) <= 100 * n * EPS
    for _ in range(3):
        again, it2, be2, _ = rbt.solve_batched(plan, Ad, Bd, seed=7)
        assert all(torch.equal(a, b) for a, b in zip(first, again))
        assert torch.equal(iters, it2) and torch.equal(berr, be2)


def test_team_falls_back_to_fp64(rbt):
    ns = [800, 520]
    As = [workloads.randn_matrix(n, seed=n) for n in ns]
    Bs = [workloads.randn(n, 2, seed=n) for n in ns]
    plan = rbt.batched_plan(ns, [2, 2], depth=2, prec=rbt.RBT_BF16)
    args = rbt.BatchArgs(plan, [dev(a) for a in As], [dev(b) for b in Bs])
    rbt.solve_batched_launch(plan, args, seed=5)
    assert (host(args.path) == 1).all()
    for s, (n, A, B) in enumerate(zip(ns, As, Bs)):
        assert float(args.berr[s]) <= 10 * n * EPS
        # the backward error bounds the error by the condition number
        bound = 10 * np.linalg.cond(A, np.inf) * 10 * n * EPS
        assert relfro(host(args.Xs[s]), np.linalg.solve(A, B)) <= bound


def test_team_zero_pivot_info(rbt):
    """Depth 0, identity with a 2 x 2 swap at rows 700, 701: the first zero
    pivot (701, 1-based) is found by the member that owns that strip."""
    n = 900
    A = np.eye(n)
    A[700, 700] = A[701, 701] = 0.0
    A[700, 701] = A[701, 700] = 1.0
    plan = rbt.batched_plan([n], [1], depth=0, prec=rbt.RBT_FP32)
    _, _, berr, info = rbt.solve_batched(plan, [dev(A)], [dev(np.ones((n, 1)))], max_iter=3)
    assert int(info[0]) == 701
    assert not (float(berr[0]) <= 1.0)
