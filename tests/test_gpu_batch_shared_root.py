"""Root items of a plan whose problem a block of four wavefronts stages together: the orders at
which the staged arrays change (own slice, both arrays, the poles alone, none), blocks that cross
from one problem into the next, and a fixed number of lanes for which nothing is staged."""
import numpy as np
import pytest

from paper_1302_7203_amd import workloads as W
from parity import TOL, assert_close

pytestmark = pytest.mark.gpu

# arrowheads hold n - 1 poles, DPR1 n: 2 * 640 doubles are a wavefront's slice, 4 * 1280 the block's
PLANS = {
    "own_or_shared": [("arrow", 641), ("arrow", 642), ("dpr1", 640), ("dpr1", 641), ("svd", 641), ("svd", 643),
                      ("herm", 641), ("herm", 642), ("arrow", 17), ("dpr1", 1), ("arrow", 1)],
    "both_or_poles": [("arrow", 2561), ("arrow", 2562), ("dpr1", 2560), ("svd", 650), ("arrow", 33)],
    "poles_or_none": [("arrow", 5122), ("arrow", 5121), ("dpr1", 1023)],
    "small_only": [("arrow", 640), ("dpr1", 16), ("svd", 65)],
}
MAKE = {"arrow": W.uniform_arrow, "dpr1": W.dpr1, "svd": W.svd_arrow, "herm": W.herm_arrow}


@pytest.mark.parametrize("plan, lanes", [(p, 0) for p in PLANS] + [("own_or_shared", 4), ("own_or_shared", 32)])
def test_shared_and_own_items(plan, lanes):
    import torch
    from paper_1302_7203_amd import batch, binding
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(23)
    probs = [MAKE[kind](n, rng) for kind, n in PLANS[plan]]
    if lanes:
        batch.set_lanes_table([binding.INT32_MAX], [lanes], device=0)
    try:
        b = batch.Batch(probs, device=dev)
        for _ in range(2):
            b.out_pool.fill_(float("nan"))
            b.run()
    finally:
        if lanes:
            batch.set_lanes_table([], [], device=0)
            binding.apply_tuned(binding.handle(0))
    torch.cuda.synchronize(dev)
    for q, pr in enumerate(probs):
        d = torch.from_numpy(pr.d).to(dev)
        z = torch.from_numpy(pr.z).to(dev)
        if pr.kind == W.KIND_SVD:
            s = binding.arrow_svd(d, z, pr.scalar)
            lam, V = s.lam, s.V
        else:
            s = {W.KIND_ARROW: binding.arrow_eig, W.KIND_DPR1: binding.dpr1_eig,
                 W.KIND_HERM: binding.arrow_eig_herm}[pr.kind](d, z, pr.scalar)
            lam, V = s.lam, s.V
        got = b.result(q)
        # the single solve and the plan are each within TOL of the exact entries
        what = f"{PLANS[plan][q]}"
        assert_close(got[0].cpu().numpy(), lam.cpu().numpy(), what + " values", 2 * TOL)
        x, y = got[1].cpu().numpy(), V.cpu().numpy()
        if pr.kind == W.KIND_HERM:
            assert np.max(np.abs(x - y) / np.abs(y)) <= 2 * TOL
        else:
            assert_close(x, y, what + " vectors", 2 * TOL)
    b.close()
