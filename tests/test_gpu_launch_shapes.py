"""Single solves at the orders where their launches change: one block ranks up to 256
poles alone, several above, the order check's own path above 16384; one launch finishes
up to n = 1280, three above; above 4608 root stage and vectors share a launch, with poles
and weights in LDS to about n = 10150, the poles alone to about 20200, neither above.  Bars: the oracle at 1e-13 on sampled eigenpairs, and bitwise
the same result however the poles are ordered."""
import numpy as np
import pytest

import oracle
from paper_1302_7203_amd import workloads as W
from parity import assert_close

pytestmark = pytest.mark.gpu


def _solve(pr, **kw):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    d, z = torch.from_numpy(pr.d.copy()).to(dev), torch.from_numpy(pr.z.copy()).to(dev)
    f = {W.KIND_ARROW: binding.arrow_eig, W.KIND_DPR1: binding.dpr1_eig, W.KIND_SVD: binding.arrow_svd,
         W.KIND_HERM: binding.arrow_eig_herm}[pr.kind]
    out = f(d, z, pr.scalar, **kw)
    torch.cuda.synchronize(dev)
    return out


def _sampled(pr, out, vectors=True, count=8):
    ks = np.unique(np.linspace(0, pr.n - 1, min(pr.n, count)).astype(np.int64))
    if pr.kind == W.KIND_SVD:
        r = oracle.arrow_svd(pr.d, pr.z, pr.scalar, ks=ks)
        rl, rV = r.sigma, r.V
    else:
        f = {W.KIND_ARROW: oracle.arrow_eig, W.KIND_DPR1: oracle.dpr1_eig, W.KIND_HERM: oracle.herm_eig}[pr.kind]
        r = f(pr.d, pr.z, pr.scalar, ks=ks)
        rl, rV = r.lam, r.vec
    assert_close(out.lam.cpu().numpy()[ks], rl, f"kind {pr.kind} n={pr.n} values")
    if vectors:
        V = out.V[:, ks.tolist()].cpu().numpy()
        if pr.kind == W.KIND_HERM:
            assert np.max(np.abs(V - rV) / np.abs(rV)) <= 1e-13
        else:
            assert_close(V, rV, f"kind {pr.kind} n={pr.n} vectors")


def _make(kind, n, rng):
    return {W.KIND_ARROW: W.uniform_arrow, W.KIND_DPR1: W.dpr1, W.KIND_SVD: W.svd_arrow, W.KIND_HERM: W.herm_arrow}[
        kind](n, rng)


@pytest.mark.parametrize("n", [2, 64, 65, 66, 129, 256, 257, 258, 1280, 1281])
@pytest.mark.parametrize("kind", [W.KIND_ARROW, W.KIND_DPR1, W.KIND_SVD, W.KIND_HERM])
def test_orders_at_the_edges_of_the_launches(kind, n, oracle_lib):
    import torch
    rng = np.random.default_rng(1000 * kind + n)
    pr = _make(kind, n, rng)
    perm = np.argsort(-np.abs(pr.d) if kind == W.KIND_SVD else -pr.d, kind="stable")
    srt = W.Problem(kind, n, pr.d[perm], pr.z[perm], pr.scalar)
    base = _solve(srt)
    _sampled(srt, base)
    m = pr.d.size
    for q in (np.arange(m)[::-1].copy(), rng.permutation(m)):
        out = _solve(W.Problem(kind, n, srt.d[q], srt.z[q], srt.scalar))
        assert torch.equal(out.lam, base.lam) and torch.equal(out.info, base.info)
        rows = torch.from_numpy(np.concatenate([q, np.arange(m, n)])).to(base.V.device)
        assert torch.equal(out.V, base.V[rows])


@pytest.mark.parametrize("m", [16384, 16385])
def test_largest_single_launch_order(m, oracle_lib):
    import torch
    rng = np.random.default_rng(m)
    pr = W.uniform_arrow(m + 1, rng, -1e4, 1e4)
    base = _solve(pr, vectors=False)
    _sampled(pr, base, vectors=False, count=4)
    q = rng.permutation(m)
    out = _solve(W.Problem(pr.kind, pr.n, pr.d[q], pr.z[q], pr.scalar), vectors=False)
    assert torch.equal(out.lam, base.lam)


@pytest.mark.parametrize("n", [40, 300, 1300])
def test_equal_poles_and_bad_input_are_seen_in_any_order(n, oracle_lib):
    """Equal poles of a DPR1 problem and poles that are not numbers are reported, and a
    reducible arrowhead is deflated, by the block that ranks alone and by several."""
    rng = np.random.default_rng(n)
    pr = W.dpr1(n, rng)
    pr.d[n // 2] = pr.d[3]
    for q in (np.argsort(-pr.d, kind="stable"), rng.permutation(n)):
        out = _solve(W.Problem(pr.kind, n, pr.d[q], pr.z[q], pr.scalar))
        assert bool((out.info.cpu() == 16).all()) and bool(out.lam.isnan().all()) and bool(out.V.isnan().all())
    bad = W.uniform_arrow(n, rng)
    bad.d[5] = np.nan
    out = _solve(bad)
    assert bool((out.info.cpu() == 32).all()) and bool(out.lam.isnan().all())
    bad.d[7] = bad.d[2]          # an equal pair beside it
    assert bool((_solve(bad).info.cpu() == 48).all())
    red = W.reducible_arrow(n, rng, zero_frac=0.3, repeat_every=4)
    out = _solve(red)
    ref = oracle.arrow_eig(red.d, red.z, red.scalar, ks=np.arange(0, n, max(1, n // 40)))
    ks = np.arange(0, n, max(1, n // 40))
    assert_close(out.lam.cpu().numpy()[ks], ref.lam, "reducible values")
    assert_close(out.V.cpu().numpy()[:, ks], ref.vec, "reducible vectors")
    assert np.array_equal((out.info.cpu().numpy()[ks] & 1024) != 0, ref.tau == 0)


@pytest.mark.parametrize("kind,n", [(W.KIND_ARROW, 4608), (W.KIND_ARROW, 4609), (W.KIND_DPR1, 4613), (W.KIND_SVD, 4610),
                                    (W.KIND_HERM, 4611), (W.KIND_DPR1, 5000), (W.KIND_SVD, 8193),
                                    (W.KIND_ARROW, 10100), (W.KIND_DPR1, 10101), (W.KIND_ARROW, 10240)])
def test_large_problems_in_any_order(kind, n, oracle_lib):
    import torch
    rng = np.random.default_rng(7000 * kind + n)
    pr = _make(kind, n, rng)
    if kind == W.KIND_DPR1 and n % 2:
        pr.scalar = -pr.scalar
    perm = np.argsort(-np.abs(pr.d) if kind == W.KIND_SVD else -pr.d, kind="stable")
    srt = W.Problem(kind, n, pr.d[perm], pr.z[perm], pr.scalar)
    base = _solve(srt)
    # the first and last eigenvalues of the blocks (of at least 16) among the samples
    _sampled(srt, base, count=40)
    assert not bool(base.V.isnan().any())
    q = rng.permutation(pr.d.size)
    out = _solve(W.Problem(kind, n, srt.d[q], srt.z[q], srt.scalar))
    assert torch.equal(out.lam, base.lam) and torch.equal(out.info, base.info)
    rows = torch.from_numpy(np.concatenate([q, np.arange(q.size, n)])).to(base.V.device)
    assert torch.equal(out.V, base.V[rows])
    vals = _solve(srt, vectors=False)
    assert torch.equal(vals.lam, base.lam) and torch.equal(vals.info, base.info)


@pytest.mark.parametrize("n", [3001, 5000])
def test_large_reducible_and_clustered(n, oracle_lib):
    rng = np.random.default_rng(n)
    red = W.reducible_arrow(n, rng, zero_frac=0.2, repeat_every=7)
    out = _solve(red)
    ks = np.arange(0, n, max(1, n // 60))
    ref = oracle.arrow_eig(red.d, red.z, red.scalar, ks=ks)
    assert_close(out.lam.cpu().numpy()[ks], ref.lam, "reducible values")
    assert_close(out.V.cpu().numpy()[:, ks], ref.vec, "reducible vectors")
    assert not bool(out.V.isnan().any())
    srt = np.argsort(-red.d, kind="stable")          # presented in order: the deflated rows stay the caller's
    out2 = _solve(W.Problem(red.kind, n, red.d[srt], red.z[srt], red.scalar))
    assert np.array_equal(out2.lam.cpu().numpy(), out.lam.cpu().numpy())
    grd = W.graded_arrow(n, rng, clusters=40)
    out = _solve(grd)
    flagged = np.nonzero(out.info.cpu().numpy() & 6)[0]
    assert flagged.size > 20
    ks = np.unique(np.concatenate([ks, flagged[:: max(1, flagged.size // 40)]]))
    ref = oracle.arrow_eig(grd.d, grd.z, grd.scalar, ks=ks)
    assert_close(out.lam.cpu().numpy()[ks], ref.lam, "graded values")
    assert_close(out.V.cpu().numpy()[:, ks], ref.vec, "graded vectors")


def test_larger_than_the_staged_poles(oracle_lib):
    rng = np.random.default_rng(9)
    pr = W.uniform_arrow(20500, rng, -1e4, 1e4)
    out = _solve(pr, vectors=False)
    _sampled(pr, out, vectors=False, count=4)


def test_deflated_beside_repaired_eigenvalues(oracle_lib):
    """Deflated values next to eigenvalues that a repair moves: a zero pole with a zero
    shaft entry beside an eigenvalue far below the first pass's resolution (either sign),
    and unit vectors inside tight clusters."""
    for alpha in (1e-30, -1e-30, 1e-12):
        d = np.array([1.0, 0.0, -1.0, 0.5, 0.5, -0.25])
        z = np.array([1.0, 0.0, 1.0, 0.0, 0.0, 0.0])
        pr = W.Problem(W.KIND_ARROW, 7, d, z, alpha)
        out = _solve(pr)
        ref = oracle.arrow_eig(d, z, alpha)
        assert_close(out.lam.cpu().numpy(), ref.lam, f"alpha {alpha} values")
        assert_close(out.V.cpu().numpy(), ref.vec, f"alpha {alpha} vectors")
        assert np.array_equal((out.info.cpu().numpy() & 1024) != 0, ref.tau == 0)
    rng = np.random.default_rng(31)
    pr = W.graded_arrow(700, rng, clusters=60)
    pr.z[rng.choice(699, 150, replace=False)] = 0.0
    out = _solve(pr)
    ref = oracle.arrow_eig(pr.d, pr.z, pr.scalar)
    assert_close(out.lam.cpu().numpy(), ref.lam, "clusters: values")
    assert_close(out.V.cpu().numpy(), ref.vec, "clusters: vectors")
    assert np.array_equal((out.info.cpu().numpy() & 1024) != 0, ref.tau == 0)


@pytest.mark.parametrize("n", [4608, 4609, 10200])
def test_pairs_keep_the_tuned_lanes(n, oracle_lib):
    """With pairs asked for every order runs the root kernel of the tuned lane count, which the
    lanes option picks above 4608 for calls without them: bitwise one result, and shift + mu = lambda."""
    import torch
    from paper_1302_7203_amd import binding
    pr = W.graded_arrow(n, np.random.default_rng(n))
    out = _solve(pr, vectors=False, pairs=True)
    _sampled(pr, out, vectors=False, count=4)
    lam = (out.shift + out.mu).cpu().numpy()
    assert np.all(np.abs(lam - out.lam.cpu().numpy()) <= 2.0 ** -52 * np.abs(lam))
    if n > 4608:
        lanes = [g for m, g in zip(*binding.read_tuned()["single"]) if n <= m][0]
        binding.set_option(binding.OPT_LANES, lanes)
        try:
            same = _solve(pr, vectors=False)
        finally:
            binding.set_option(binding.OPT_LANES, 0)
        assert torch.equal(same.lam, out.lam)
