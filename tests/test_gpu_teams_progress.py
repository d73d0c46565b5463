"""Teams of the batched solver whose workgroups do not wait for each other to
start (a limit of 0) give the same bits; where every wait expires (a negative
limit) the systems with teams report NaN and the launch ends."""
import pytest
import torch

from paper_2312_09376_amd import _lib, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rbt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_09376_amd import rbt as r
    r.lib()
    return r


def test_spin_limits(rbt):
    ns, ks = [1500, 900, 600, 100], [2, 1, 3, 1]
    plan = rbt.batched_plan(ns, ks, depth=2, prec=rbt.RBT_FP32)
    As = [workloads.device_shifted(n, n) for n in ns]
    Bs = [workloads.device_randn(n, k, n) for n, k in zip(ns, ks)]
    args = rbt.BatchArgs(plan, As, Bs)

    def run(limit):
        default = rbt.get_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT)
        rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, limit)
        try:
            rbt.solve_batched_launch(plan, args, seed=5)
            torch.cuda.synchronize()
        finally:
            rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, default)
        return [x.clone() for x in args.Xs], args.berr.clone()

    X, berr = run(1 << 20)
    assert bool(torch.isfinite(berr).all())
    X0, berr0 = run(0)
    assert all(torch.equal(a, b) for a, b in zip(X, X0)) and torch.equal(berr, berr0)
    Xn, berrn = run(-1)
    assert all(bool(torch.isnan(x).all()) for x in Xn[:3]) and bool(torch.isnan(berrn[:3]).all())
    assert torch.equal(Xn[3], X[3])  # (no team: no wait)
    X1, _ = run(1 << 20)
    assert all(torch.equal(a, b) for a, b in zip(X, X1))
