"""The inverses of a diagonal block that the batched solver's FP64 fallback
multiplies by without a refinement step must be as accurate as substitution by
columns: |D X - I| <= gamma |D| |X| componentwise, gamma = 2 n eps for sums of at
most n products and a division. Unpivoted N(0,1) blocks, whose 16 x 16 diagonal
tiles are ill conditioned: there a tile's product with its own explicit inverse
exceeds the bound."""
import os
import struct

import numpy as np
import pytest

from paper_2312_09376_amd import workloads

E = pytest.importorskip("tests.hostemu.emu_blocks")
EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def exe():
    if E.emu.clang() is None:
        pytest.skip("clang++ not available")
    return E.build(exe=os.path.join(E.emu.OUT_DIR, "emu_batched_diag"), sources=[],
                   driver="emu_batched_diag.cpp", watch=["k_batched.hip"])


@pytest.mark.parametrize("n", [64, 50, 17])
@pytest.mark.parametrize("seed", range(8))
def test_inverses_have_the_residual_of_substitution(exe, n, seed):
    A = workloads.randn_matrix(n, seed=100 * n + seed)
    raw = E.run(exe, struct.pack("<q", n) + np.asfortranarray(A).tobytes(order="F"))
    F = np.frombuffer(raw, np.float64, n * n).reshape(n, n, order="F")
    W = np.frombuffer(raw, np.float64, 64 * 64, 8 * n * n).reshape(64, 64, order="F")[:n, :n]
    eye = np.eye(n)
    for D, X in ((np.tril(F, -1) + eye, np.tril(W, -1) + eye), (np.triu(F), np.triu(W))):
        R = np.abs(D.astype(np.longdouble) @ X.astype(np.longdouble) - eye)
        assert (R <= 2 * n * EPS * (np.abs(D) @ np.abs(X))).all()
