"""The check stage's lists in a plan of many small problems: every eigenvalue listed (the
bisection leaves no norm, so each needs a pass), more than a block gathers; repairs and
deflations among problems that list nothing."""
import numpy as np
import pytest

import near_zero_cases as NZ
import oracle
from paper_1302_7203_amd import workloads as W
from parity import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("root", ["bisect", "rational"])
def test_lists_of_many_small_problems(root, oracle_lib):
    import torch
    from paper_1302_7203_amd import batch, binding
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(17)
    kinds = [W.uniform_arrow(64, rng), W.dpr1(64, rng), W.svd_arrow(64, rng), W.herm_arrow(63, rng),
             W.reducible_arrow(60, rng, zero_frac=0.3, repeat_every=5), W.uniform_arrow(1, rng)]
    _, d, z, a = NZ.arrow_cases()[0]
    kinds.append(W.Problem(W.KIND_ARROW, d.size + 1, d, z, a))
    probs = [kinds[p % len(kinds)] for p in range(17000)]
    if root == "bisect":
        binding.set_option(binding.OPT_ROOT, binding.ROOT_BISECT)
    try:
        b = batch.Batch(probs, device=dev)
    finally:
        binding.set_option(binding.OPT_ROOT, binding.ROOT_RATIONAL)
    b.out_pool.fill_(float("nan"))
    for _ in range(2):
        b.run()
    torch.cuda.synchronize(dev)
    for q, pr in enumerate(kinds):
        first = b.result(q)
        if pr.kind == W.KIND_SVD:
            r = oracle.arrow_svd(pr.d, pr.z, pr.scalar)
            rl, rV = r.sigma, r.V
            assert_close(first[2].cpu().numpy(), r.U, "left vectors")
        else:
            f = {W.KIND_ARROW: oracle.arrow_eig, W.KIND_DPR1: oracle.dpr1_eig, W.KIND_HERM: oracle.herm_eig}[pr.kind]
            r = f(pr.d, pr.z, pr.scalar)
            rl, rV = r.lam, r.vec
        assert_close(first[0].cpu().numpy(), rl, f"problem {q} values")
        V = first[1].cpu().numpy()
        if pr.kind == W.KIND_HERM:
            assert np.max(np.abs(V - rV) / np.abs(rV)) <= 1e-13
        else:
            assert_close(V, rV, f"problem {q} vectors")
        for p in range(q + len(kinds), len(probs), 11 * len(kinds)):      # the same bits wherever it stands
            for x, y in zip(b.result(p), first):
                assert (x is None) == (y is None) and (x is None or torch.equal(x, y)), (p, q)
    b.close()
