"""The slab kernel of the elimination with partial pivoting (k_gepp.hip) as host
C++ under AddressSanitizer: the exchange between workgroups that run at once, and
what happens when they do not all run, as on a device that other work keeps
busy: one of them factors the slab, with the same pivots, and nothing waits for
good."""
import os
import struct

import numpy as np
import pytest

from oracle import pivoted
from paper_2312_09376_amd import workloads

E = pytest.importorskip("tests.hostemu.emu_blocks")
EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def exe():
    if E.emu.clang() is None:
        pytest.skip("clang++ not available")
    return E.build(exe=os.path.join(E.emu.OUT_DIR, "emu_gepp"), sources=["k_gepp.hip", "k_trsm.hip"],
                   driver="emu_gepp.cpp")


def gepp(exe, A, limit, threads):
    n = A.shape[0]
    raw = E.run(exe, struct.pack("<2q", n, limit) + np.asfortranarray(A).tobytes(order="F"),
                env={"EMU_THREADS": str(threads)})
    LU = np.frombuffer(raw, np.float64, n * n).reshape(n, n, order="F")
    ipiv = np.frombuffer(raw, np.int64, n, 8 * n * n)
    perm = np.frombuffer(raw, np.int64, n, 8 * n * n + 8 * n)
    info, err = struct.unpack("<2i", raw[-8:])
    return LU, ipiv, perm, info, err


def check(exe, A, limit, threads, info=0):
    n = A.shape[0]
    LU, ipiv, perm, got_info, err = gepp(exe, A, limit, threads)
    LUo, ipiv_o, info_o = pivoted.gepp(A)
    assert got_info == info_o == info and err == 0
    k = n if info == 0 else info - 1
    assert np.array_equal(ipiv[:k], ipiv_o[:k])
    L = np.tril(LUo, -1) + np.eye(n)
    den = np.abs(L[:, :k]) @ np.abs(np.triu(LUo)[:k, :k])
    assert (np.abs(LU[:, :k] - LUo[:, :k]) <= 4 * n * EPS * den + 1e-300).all()
    want = np.arange(n)
    for j, p in enumerate(ipiv - 1):
        want[[j, p]] = want[[p, j]]
    assert np.array_equal(perm, want)


# 1100 rows: three workgroups in the first slabs, two from 1024 rows down (one)
@pytest.mark.parametrize("limit,threads", [(1 << 20, 4), (50, 1), (50, 2), (0, 4)])
def test_slabs_with_all_and_with_few_workgroups_running(exe, limit, threads):
    check(exe, workloads.randn_matrix(1100, seed=5), limit, threads)


@pytest.mark.parametrize("limit,threads", [(50, 1)])
def test_zero_column(exe, limit, threads):
    A = workloads.randn_matrix(1060, seed=6)
    A[:, 20] = 0.0
    check(exe, A, limit, threads, info=21)


def test_negative_limit_leaves_no_finite_slab(exe):
    LU, _, _, info, err = gepp(exe, workloads.randn_matrix(1100, seed=5), -1, 4)
    assert err == 1 and info == -1
    assert np.isnan(LU[:, :32]).all()
