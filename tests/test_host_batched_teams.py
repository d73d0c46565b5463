"""Teams of workgroups in the host build of the batched solver (tests/hostemu,
AddressSanitizer): a system of order 512 solved by a team of 8 gives bit for bit what
one workgroup gives, whether the team's workgroups all run at once, cannot (fewer
host threads than members) or do not wait for each other; where every wait
expires (forced by a negative limit) the result is NaN, and the launch ends."""
import numpy as np
import pytest

from paper_2312_09376_amd import workloads

emu = pytest.importorskip("tests.hostemu.emu")

EPS = 2.0 ** -52
FP32 = 1  # RBT_FP32


@pytest.fixture(scope="module")
def exe():
    if emu.clang() is None:
        pytest.skip("clang++ not available")
    return emu.build()


@pytest.fixture(scope="module")
def batch():
    ns, ks = [520, 40], [2, 1]
    As = [workloads.dominant(n, seed=n) for n in ns]
    Bs = [workloads.randn(n, k, seed=n + 1) for n, k in zip(ns, ks)]
    return As, Bs


def run(batch, grid, threads, spin_limit=None):
    As, Bs = batch
    out = emu.run_batched(As, Bs, depth=2, prec=FP32, seed=7, max_iter=10, grid=grid, threads=threads,
                          spin_limit=spin_limit)
    checks = out[5]
    assert checks["plan_intact"] and checks["divergent_barriers"] == 0
    # one ticket for the small system; four members' or, without teams, one for the large one
    return out, checks["ticket"] - grid - 1


@pytest.fixture(scope="module")
def alone(exe, batch):
    out, large = run(batch, 2, 2)
    assert large == 1
    for A, B, X, be in zip(*batch, out[0], out[2]):
        assert be <= 10 * A.shape[0] * EPS
        assert np.linalg.norm(X - np.linalg.solve(A, B)) <= 100 * A.shape[0] * EPS * np.linalg.norm(X)
    return out


@pytest.mark.parametrize("threads,spin_limit", [(8, None), (2, 20), (8, 0)])
def test_a_team_gives_what_one_workgroup_gives(batch, alone, threads, spin_limit):
    out, large = run(batch, 8, threads, spin_limit)
    assert large == 4  # a team of four: an order below 1024
    assert all(np.array_equal(x, y) for x, y in zip(out[0], alone[0]))
    for a, b in zip(out[1:5], alone[1:5]):
        assert np.array_equal(a, b)


def test_expired_waits_report_nan(batch, alone):
    out, _ = run(batch, 8, 8, spin_limit=-1)
    assert np.isnan(out[0][0]).all() and np.isnan(out[2][0])
    assert np.array_equal(out[0][1], alone[0][1])  # the small system has no team
