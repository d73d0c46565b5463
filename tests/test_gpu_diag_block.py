"""The diagonal-block kernel at every remainder class: orders of one block
around its 16-column steps and its 64-row wavefronts, and one past it. The
factors must reproduce the matrix within the elimination's own rounding
bound, |A - L U| <= 2 n eps |L| |U| in every entry, and a zero pivot must be
reported at its place in any step."""
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


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 33, 48, 63, 65, 79, 80, 81, 97, 112, 113, 127,
                               128, 129, 145])
@pytest.mark.parametrize("pad", [0, 3])
def test_reproduces_the_matrix(rbt, n, pad):
    A = workloads.randn_matrix(n, seed=n) + 2.0 * np.eye(n)
    buf = torch.zeros(n, n + pad, dtype=torch.float64, device="cuda")
    Ad = buf.t()[:n]  # column-major, leading dimension n + pad
    Ad.copy_(torch.from_numpy(A))
    LU, info = rbt.genp(Ad)
    F = LU.cpu().numpy()
    L = np.tril(F, -1) + np.eye(n)
    U = np.triu(F)
    err = np.abs(A.astype(np.longdouble) - L.astype(np.longdouble) @ U.astype(np.longdouble))
    assert int(info) == 0
    assert (err <= 2 * n * EPS * (np.abs(L) @ np.abs(U))).all()
    assert not buf[:, n:].any()  # nothing written beyond the matrix


@pytest.mark.parametrize("col", [1, 16, 17, 32, 100, 127, 128])
def test_zero_pivot_position(rbt, col):
    d = np.ones(128)
    d[col - 1] = 0.0
    _, info = rbt.genp(dev(np.diag(d)))
    assert int(info) == col
