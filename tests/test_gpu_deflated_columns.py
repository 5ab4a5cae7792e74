"""Columns of deflated eigenpairs beside eigenvalues that a remedy of Remark 2 moves far from
their first-pass value: every column is written once, by single solves on every path and by
plans, and the pairs are the oracle's."""
import numpy as np
import pytest

import deflated_cases as C
import oracle
from paper_1302_7203_amd import workloads as W
from parity import assert_close

pytestmark = pytest.mark.gpu

DEFLATED = 1024


def _solve(pr, vectors=True):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    out = binding.arrow_eig(torch.from_numpy(pr.d).to(dev), torch.from_numpy(pr.z).to(dev), pr.scalar, vectors=vectors)
    torch.cuda.synchronize(dev)
    return out


def _check(pr, lam, V, info, what):
    ks = np.arange(pr.n) if pr.n <= 400 else np.unique(np.concatenate(
        [np.arange(0, pr.n, pr.n // 60), np.nonzero(info & 6)[0][:60], np.nonzero(info & DEFLATED)[0][:60]]))
    ref = oracle.arrow_eig(pr.d, pr.z, pr.scalar, ks=ks)
    assert_close(lam[ks], ref.lam, what + " values")
    assert np.array_equal((info[ks] & DEFLATED) != 0, ref.tau == 0), what
    if V is not None:
        assert_close(V[:, ks], ref.vec, what + " vectors")
    # all columns: in descending order, as many deflated ones as the input has
    assert np.all(lam[:-1] >= lam[1:]), what
    poles, count = np.unique(pr.d[pr.z != 0.0], return_counts=True)
    assert np.count_nonzero(info & DEFLATED) == pr.d.size - poles.size, what


def _widened(pr):
    """`pr` and `pr` with rows between first-pass and final values."""
    from paper_1302_7203_amd import binding
    yield "", pr
    final = _solve(pr, vectors=False)
    binding.set_option(binding.OPT_REMEDIES, 0)
    try:
        first = _solve(pr, vectors=False)
    finally:
        binding.set_option(binding.OPT_REMEDIES, 1)
    lam = [o.lam.cpu().numpy()[(o.info.cpu().numpy() & DEFLATED) == 0] for o in (first, final)]
    wide = C.between(pr, *lam, most=min(24, 1280 - pr.n) if pr.n <= 1280 else 24)
    if wide.n > pr.n:
        yield ", rows between", wide


@pytest.mark.parametrize("name, pr", C.cases(), ids=[n for n, _ in C.cases()])
def test_single_solves(name, pr, oracle_lib):
    for more, q in _widened(pr):
        for vectors in (True, False):
            out = _solve(q, vectors)
            _check(q, out.lam.cpu().numpy(), out.V.cpu().numpy() if vectors else None, out.info.cpu().numpy(),
                   name + more)


@pytest.mark.parametrize("n", [1500, 4800])
def test_larger_single_solves(n, oracle_lib):
    rng = np.random.default_rng(n)
    pr = W.graded_arrow(n, rng, clusters=n // 14)
    pr.z[rng.choice(n - 1, n // 5, replace=False)] = 0.0
    for more, q in _widened(pr):
        out = _solve(q)
        _check(q, out.lam.cpu().numpy(), out.V.cpu().numpy(), out.info.cpu().numpy(), f"graded {n}" + more)


def test_plan(oracle_lib):
    import torch
    from paper_1302_7203_amd import batch
    dev = torch.device("cuda", 0)
    probs = [q for _, pr in C.cases() for _, q in _widened(pr)]
    b = batch.Batch(probs, device=dev)
    b.out_pool.fill_(float("nan"))
    b.run()
    torch.cuda.synchronize(dev)
    for p, q in enumerate(probs):
        lam, V, _, info = b.result(p)
        _check(q, lam.cpu().numpy(), V.cpu().numpy(), info.cpu().numpy(), f"problem {p}, n {q.n}")
    b.close()
