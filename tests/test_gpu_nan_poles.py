"""Poles that are not numbers: equal poles beside them are still seen, whatever an earlier problem
left in the workspace, and the report takes about as long as a solve."""
import numpy as np
import pytest

from paper_1302_7203_amd import workloads as W

pytestmark = pytest.mark.gpu

NONFINITE, REDUCIBLE = 32, 16
MAKE = {W.KIND_ARROW: W.uniform_arrow, W.KIND_DPR1: W.dpr1, W.KIND_SVD: W.svd_arrow, W.KIND_HERM: W.herm_arrow}


def _solve(pr, vectors=False):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    f = {W.KIND_ARROW: binding.arrow_eig, W.KIND_DPR1: binding.dpr1_eig, W.KIND_SVD: binding.arrow_svd,
         W.KIND_HERM: binding.arrow_eig_herm}[pr.kind]
    return f(torch.from_numpy(pr.d.copy()).to(dev), torch.from_numpy(pr.z.copy()).to(dev), pr.scalar, vectors=vectors)


@pytest.mark.parametrize("kind", list(MAKE))
@pytest.mark.parametrize("n", [3, 66, 257, 300, 2100])
def test_equal_poles_beside_nan(kind, n):
    rng = np.random.default_rng(n + kind)
    clean = MAKE[kind](n, rng)
    m = clean.d.size
    equal = W.Problem(kind, n, rng.permutation(clean.d), clean.z, clean.scalar)
    equal.d[0] = equal.d[m - 1]
    for count in sorted({1, m // 3, m - 2, m - 1, m} - {0}):
        for src, flag in ((clean, 0), (equal, REDUCIBLE)):
            if not 1 <= count <= m - 2 and src is equal:
                continue
            before = _solve(clean if src is equal else equal)   # leaves equal entries, or none, behind
            pr = W.Problem(kind, n, src.d.copy(), src.z, src.scalar)
            pr.d[1 + rng.choice(m - 2, count, replace=False) if count <= m - 2 else np.arange(m - count, m)] = np.nan
            out = _solve(pr, vectors=True)
            assert bool((out.info.cpu() == (NONFINITE | flag)).all()), (count, flag)
            assert bool(out.lam.isnan().all()) and bool(out.V.isnan().all())
            del before


def test_report_is_not_slower_than_a_solve():
    import torch
    rng = np.random.default_rng(1)
    pr = W.uniform_arrow(16000, rng)
    pr.d = rng.permutation(pr.d)
    bad = W.Problem(pr.kind, pr.n, pr.d.copy(), pr.z, pr.scalar)
    bad.d[5000] = np.nan
    best = {}
    for name, q in (("solve", pr), ("report", bad)):
        _solve(q)
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            _solve(q)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        best[name] = min(times)
    assert best["report"] <= best["solve"], best
