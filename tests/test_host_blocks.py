"""The elimination's block kernels (k_getrf.hip, k_trsm.hip) as host C++ under
AddressSanitizer, work-items as fibers (tests/hostemu): what they compute may
not depend on how far one wavefront runs ahead of another between barriers."""
import numpy as np
import pytest

from paper_2312_09376_amd import workloads

E = pytest.importorskip("tests.hostemu.emu_blocks")


@pytest.fixture(scope="module")
def exe():
    if E.emu.clang() is None:
        pytest.skip("clang++ not available")
    return E.build()


@pytest.mark.parametrize("op,dt", [(0, np.float64), (1, np.float32), (2, np.float32)])
@pytest.mark.parametrize("n", [16, 33, 100, 128])
def test_diag_block_in_any_wavefront_order(exe, op, dt, n):
    """In turn, each wavefront as far as it can go, and the same from the last
    one: bit-identical factors, which reproduce the matrix."""
    A = (workloads.randn_matrix(n, seed=n) + 2 * np.eye(n)).astype(dt)
    F = [E.call(exe, op, A, order=o)[0] for o in (0, 1, 2)]
    assert np.array_equal(F[0], F[1]) and np.array_equal(F[0], F[2])
    L = np.tril(F[0], -1).astype(float) + np.eye(n)
    U = np.triu(F[0]).astype(float)
    assert (np.abs(A - L @ U) <= 2 * n * np.finfo(dt).eps * (np.abs(L) @ np.abs(U))).all()
