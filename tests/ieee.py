"""Plain substitution with IEEE Inf and NaN as they come, and the comparison with
it, for the tests of triangular solves beside a zero pivot."""
import numpy as np

from paper_2312_09376_amd import workloads


def substitution(T, B, lower, unit):
    """op(T) X = B entry by entry in the arrays' type, a division by a pivot as
    a product with its reciprocal; IEEE Inf and NaN as they come."""
    X = B.copy()
    n = T.shape[0]
    one = T.dtype.type(1)
    with np.errstate(all="ignore"):
        for j in (range(n) if lower else range(n - 1, -1, -1)):
            if not unit:
                X[j] = X[j] * (one / T[j, j])
            rows = slice(j + 1, n) if lower else slice(0, j)
            X[rows] -= np.outer(T[rows, j], X[j])
    return X


def same_nonfinite(got, want):
    """NaN where NaN and the same infinities; finite entries within the bound
    of the elimination's own rounding on well conditioned data."""
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf])
    fin = np.isfinite(want)  # (none where the first pivot solved is the zero)
    eps = np.finfo(want.dtype).eps
    top = np.abs(want[fin]).max(initial=1.0)
    assert np.abs(got[fin] - want[fin]).max(initial=0.0) <= 1000 * eps * top


def tame(n, dt, seed=3):
    """A matrix whose triangles are well conditioned."""
    return (0.05 * workloads.randn_matrix(n, seed=seed) + np.eye(n)).astype(dt)
