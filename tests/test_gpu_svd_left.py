"""Left singular vectors by every vector launch of single solves, one and two rows a store: against
the oracle, and u_r = sigma v_r / d_r from the vectors returned."""
import numpy as np
import pytest

import oracle
from paper_1302_7203_amd import workloads as W
from parity import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 65, 257, 258, 778, 1280, 1281, 1282, 2049, 4100, 4610])
def test_left_vectors(n, oracle_lib):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    pr = W.svd_arrow(n, np.random.default_rng(n))
    d, z = torch.from_numpy(pr.d).to(dev), torch.from_numpy(pr.z).to(dev)
    out = binding.arrow_svd(d, z, pr.scalar)
    torch.cuda.synchronize(dev)
    ks = np.unique(np.linspace(0, n - 1, min(n, 12)).astype(int))
    ref = oracle.arrow_svd(pr.d, pr.z, pr.scalar, ks=ks)
    assert_close(out.U[:, ks.tolist()].cpu().numpy(), ref.U, f"n={n} left vectors")
    assert torch.equal(out.U[:-1], out.lam[None, :] * out.V[:-1] / d[:, None])
    assert torch.equal(out.U[-1], pr.scalar * out.V[-1] / out.lam)
