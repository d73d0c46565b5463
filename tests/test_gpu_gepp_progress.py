"""The slab kernel's workgroups need each other: where they do not come together
within the spin limit, one of them factors the slab, and the factors are the
same bit for bit; also beside other work on the device."""
import numpy as np
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


@pytest.mark.parametrize("n", [1040, 1700])
def test_no_patience_gives_the_same_factors(rbt, n):
    """A limit of 0: a workgroup that does not find every candidate at its first
    look calls the slab off. The factors do not depend on who takes it."""
    A = workloads.device_randn(n, n, n)
    LU, ipiv, info = rbt.gepp(A.clone())
    default = rbt.get_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT)
    rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, 0)
    try:
        LU0, ipiv0, info0 = rbt.gepp(A.clone())
        torch.cuda.synchronize()
    finally:
        rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, default)
    assert int(info) == int(info0) == 0
    assert torch.equal(ipiv, ipiv0) and torch.equal(LU, LU0)


def test_negative_limit_is_reported(rbt):
    """Every wait expires at once: NaN and info = -1, never a finite factor."""
    A = workloads.device_randn(1200, 1200, 4)
    default = rbt.get_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT)
    rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, -1)
    try:
        LU, _, info = rbt.gepp(A)
        torch.cuda.synchronize()
    finally:
        rbt.set_option(_lib.RBT_OPT_SWEEP_SPIN_LIMIT, default)
    assert int(info) == -1 and bool(torch.isnan(LU[:, :32]).all())


def test_beside_other_streams(rbt):
    """Three factorizations and a batch with teams at once, each on its own
    stream: the results of each by itself."""
    ns = [2600, 3000, 3400]
    As = [workloads.device_randn(n, n, n) for n in ns]
    want = [rbt.gepp(a.clone()) for a in As]
    bn, bk = [1400, 1200, 700, 300], [2, 1, 3, 1]
    plan = rbt.batched_plan(bn, bk, depth=2, prec=rbt.RBT_FP32)
    Ab = [torch.from_numpy(np.asfortranarray(workloads.dominant(n, seed=n)).T.copy()).cuda().t() for n in bn]
    Bb = [workloads.device_randn(n, k, 3) for n, k in zip(bn, bk)]
    args = rbt.BatchArgs(plan, Ab, Bb)
    rbt.solve_batched_launch(plan, args, seed=5)
    torch.cuda.synchronize()
    Xb = [x.clone() for x in args.Xs]
    copies = [a.clone() for a in As]
    works = [torch.empty(rbt.workspace_size(n, 0, 0), dtype=torch.uint8, device="cuda") for n in ns]
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    got = []
    with torch.cuda.stream(streams[3]):
        rbt.solve_batched_launch(plan, args, seed=5)
    for a, w, s in zip(copies, works, streams):
        with torch.cuda.stream(s):
            got.append(rbt.gepp(a, work=w))
    torch.cuda.synchronize()
    for (LU, ipiv, info), (LUw, ipivw, _) in zip(got, want):
        assert int(info) == 0 and torch.equal(ipiv, ipivw) and torch.equal(LU, LUw)
    assert all(torch.equal(x, y) for x, y in zip(args.Xs, Xb))
