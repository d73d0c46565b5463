"""The elimination's block kernels (k_getrf.hip, k_trsm.hip) as host C++ under
AddressSanitizer, work-items as fibers (tests/hostemu): what they compute may
not depend on how far one wavefront runs ahead of another between barriers."""
import numpy as np
import pytest

from paper_2312_09376_amd import workloads
from tests.ieee import same_nonfinite, substitution, tame

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


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("mode", [E.LN, E.UN, E.UT, E.LT])
@pytest.mark.parametrize("n,at", [(128, 37), (100, 64), (40, 39), (128, 0)])
def test_left_solve_keeps_entries_beside_a_zero_pivot(exe, f32, mode, n, at):
    """Non-unit triangles with an exact zero on the diagonal (unit ones: an
    infinite right-hand side entry): the entries solved before it, in its own
    16-row tile too, are those of plain substitution, and so are the others."""
    dt = np.float32 if f32 else np.float64
    A = tame(n, dt)
    B = workloads.randn(n, 5, seed=4).astype(dt)
    unit = mode in (E.LN, E.LT)
    if unit:
        B[at, 2] = np.inf
        T = np.tril(A, -1) + np.eye(n, dtype=dt)
    else:
        A[at, at] = 0.0
        T = np.triu(A)
    T = T.T if mode in (E.UT, E.LT) else T
    X = E.call(exe, (20 if f32 else 10) + mode, A, B)[1]
    same_nonfinite(X, substitution(np.asarray(T, dt), B, mode in (E.LN, E.UT), unit))


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("at", [5, 70])
def test_panel_solves_keep_entries_beside_a_zero_pivot(exe, f32, at):
    """L21 U11 = A21: the columns before the zero pivot are correct factors."""
    dt = np.float32 if f32 else np.float64
    m, n = 96, 100
    A = tame(m, dt)
    A[at, at] = 0.0
    B = workloads.randn(n, m, seed=5).astype(dt)
    C = workloads.randn(n, n, seed=6).astype(dt)
    C[at, 3] = np.nan
    _, X, Y, _ = E.call(exe, 31 if f32 else 30, A, B, C)
    U, L = np.triu(A), np.tril(A, -1) + np.eye(m, dtype=dt)
    same_nonfinite(X, substitution(U.T, B.T.copy(), True, False).T)
    same_nonfinite(Y[:m], substitution(L, C[:m], True, True))


def test_inverse_of_a_block_with_a_zero_pivot(exe):
    n, at = 128, 50
    A = tame(n, np.float64)
    A[at, at] = 0.0
    W = E.call(exe, 40, A)[2].reshape(2, n, n).transpose(0, 2, 1)
    same_nonfinite(W[1], substitution(np.triu(A), np.eye(n), False, False))


@pytest.mark.parametrize("op,dt", [(0, np.float64), (1, np.float32)])
@pytest.mark.parametrize("n,at", [(128, 3), (128, 20), (100, 47), (60, 33)])
def test_diag_block_keeps_rows_above_a_zero_pivot(exe, op, dt, n, at):
    """A leading block that becomes singular at one column: the rows of U up to
    it right of its 16-column step, and all columns of L before it, are those of
    plain elimination; info names the column."""
    A = tame(n, dt)
    F = A.astype(float)
    for j in range(at):
        F[j + 1:, j] /= F[j, j]
        F[j + 1:, j + 1:] -= np.outer(F[j + 1:, j], F[j, j + 1:])
    # exact zero: row `at` of L before the column is zero, and so is its diagonal
    A[at, :at] = 0
    A[at, at] = 0
    F[at, :at] = 0
    F[at, at:] = A[at, at:]
    got, _, _, info = E.call(exe, op, A)
    assert info == at + 1
    right = 16 * (at // 16 + 1)
    same_nonfinite(got[:at + 1, right:], F[:at + 1, right:].astype(dt))
    same_nonfinite(got[:, :at], F[:, :at].astype(dt))
