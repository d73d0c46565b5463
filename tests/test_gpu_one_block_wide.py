"""17 to 384 right-hand sides of an order of one block take block solves whatever
the workspace: bit for bit what the workspace without a publication buffer gives."""
import numpy as np
import pytest
import torch

from paper_2312_09376_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rbt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_09376_amd import rbt as r
    r.lib()
    return r


@pytest.mark.parametrize("trans", [0, 1])
@pytest.mark.parametrize("n,k", [(1, 17), (50, 33), (128, 384)])
def test_one_block_takes_block_solves(rbt, n, k, trans):
    LU, _ = rbt.genp(torch.from_numpy(np.ascontiguousarray(workloads.dominant(n, seed=n).T)).cuda().t())
    B = workloads.device_randn(n, k, 3)
    sync = ((64 + 2 * 16 * n) * 4 + 255) // 256 * 256
    small = torch.empty(2 * 128 * 128 * 8 + sync, dtype=torch.uint8, device="cuda")
    X = rbt.getrs(LU, B.clone(), trans=trans)
    assert torch.equal(X, rbt.getrs(LU, B.clone(), trans=trans, work=small))
