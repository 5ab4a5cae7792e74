"""Bisection (ARROW_OPT_ROOT 0) at the orders where its launches change: one launch finishes up to
three times the compute units (768), three above; above 4608 root stage and vectors share one.  And a
plan whose check lists more eigenvalues than a block gathers."""
import numpy as np
import pytest

import oracle
from paper_1302_7203_amd import workloads as W
from parity import assert_close

pytestmark = pytest.mark.gpu

MAKE = {W.KIND_ARROW: W.uniform_arrow, W.KIND_DPR1: W.dpr1, W.KIND_SVD: W.svd_arrow, W.KIND_HERM: W.herm_arrow}
REF = {W.KIND_ARROW: "arrow_eig", W.KIND_DPR1: "dpr1_eig", W.KIND_SVD: "arrow_svd", W.KIND_HERM: "herm_eig"}


@pytest.fixture
def bisect():
    from paper_1302_7203_amd import binding
    binding.set_option(binding.OPT_ROOT, binding.ROOT_BISECT)
    yield
    binding.set_option(binding.OPT_ROOT, binding.ROOT_RATIONAL)


def _solve(pr, vectors):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    f = {W.KIND_ARROW: binding.arrow_eig, W.KIND_DPR1: binding.dpr1_eig, W.KIND_SVD: binding.arrow_svd,
         W.KIND_HERM: binding.arrow_eig_herm}[pr.kind]
    out = f(torch.from_numpy(pr.d).to(dev), torch.from_numpy(pr.z).to(dev), pr.scalar, vectors=vectors)
    torch.cuda.synchronize(dev)
    return out


def _close(pr, lam, V, ks, what):
    r = getattr(oracle, REF[pr.kind])(pr.d, pr.z, pr.scalar, ks=ks)
    assert_close(lam[ks], r.sigma if pr.kind == W.KIND_SVD else r.lam, what + " values")
    rV = r.V if pr.kind == W.KIND_SVD else r.vec
    if pr.kind == W.KIND_HERM:
        assert np.max(np.abs(V[:, ks] - rV) / np.abs(rV)) <= 1e-13
    else:
        assert_close(V[:, ks], rV, what + " vectors")


@pytest.mark.parametrize("kind", list(MAKE))
@pytest.mark.parametrize("n", [2, 65, 257, 768, 769, 1281, 4609])
def test_orders(kind, n, bisect, oracle_lib):
    import torch
    pr = MAKE[kind](n, np.random.default_rng(10 * n + kind))
    out, vals = _solve(pr, True), _solve(pr, False)
    assert torch.equal(out.lam, vals.lam) and torch.equal(out.info, vals.info)
    assert not bool(out.V.isnan().any())
    listed = np.nonzero(out.info.cpu().numpy() & (2 | 4 | 8 | 512))[0]
    ks = np.unique(np.concatenate([np.linspace(0, n - 1, min(n, 10)).astype(int), listed[:8]]))
    _close(pr, out.lam.cpu().numpy(), out.V.cpu().numpy(), ks, f"kind {kind} n={n}")


@pytest.mark.parametrize("n", [300, 900, 1400])
def test_reducible(n, bisect, oracle_lib):
    import torch
    pr = W.reducible_arrow(n, np.random.default_rng(n), zero_frac=0.3, repeat_every=5)
    out, vals = _solve(pr, True), _solve(pr, False)
    assert torch.equal(out.lam, vals.lam) and torch.equal(out.info, vals.info)
    ks = np.arange(0, n, n // 50)
    _close(pr, out.lam.cpu().numpy(), out.V.cpu().numpy(), ks, f"reducible n={n}")


def test_more_listed_than_a_block_gathers(oracle_lib):
    """tau_nu = 1 asks for a remedy wherever K_nu > 1: about half of the eigenvalues."""
    import torch
    from paper_1302_7203_amd import batch, binding
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(3)
    kinds = [W.uniform_arrow(64, rng), W.dpr1(64, rng), W.svd_arrow(64, rng), W.herm_arrow(64, rng)]
    probs = [kinds[p % len(kinds)] for p in range(60000)]
    binding.set_option(binding.OPT_TAU_NU, 1.0)
    try:
        b = batch.Batch(probs, device=dev)
    finally:
        binding.set_option(binding.OPT_TAU_NU, 100.0)
    b.out_pool.fill_(float("nan"))
    for _ in range(2):
        b.run()
    torch.cuda.synchronize(dev)
    info = b.info_pool.cpu().numpy()
    # 2048 blocks hold 512 entries each at most; the check has that many or fewer
    assert np.count_nonzero(info & (2 | 4)) > 2048 * 512
    for q, pr in enumerate(kinds):
        first = b.result(q)
        _close(pr, first[0].cpu().numpy(), first[1].cpu().numpy(), np.arange(64), f"problem {q}")
        for p in range(q + len(kinds), len(probs), 97 * len(kinds)):
            for x, y in zip(b.result(p), first):
                assert (x is None) == (y is None) and (x is None or torch.equal(x, y)), (p, q)
    b.close()
