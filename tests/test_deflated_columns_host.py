"""The column rule of deflated eigenpairs on the host: a permutation whatever the accuracy of the
solved eigenvalues, and the oracle's order once they are repaired, before and after the repairs."""
import numpy as np
import pytest

import deflated_cases as C
import oracle
from emu import emu
from parity import assert_close

DEFLATED = 1024


@pytest.fixture(params=["after the repairs", "before the repairs"])
def finish(request):
    emu.set_finish_check(request.param == "before the repairs")
    yield
    emu.set_finish_check(False)


def _widened(pr):
    yield pr
    lam = []
    for remedies in (0, 1):
        r = emu.solve(0, pr.d, pr.z, pr.scalar, vectors=False, remedies=remedies)
        lam.append(r["lam"][(r["info"] & DEFLATED) == 0])
    wide = C.between(pr, *lam)
    if wide.n > pr.n:
        yield wide


def _once(pr, r):
    """Every column is written (the driver's buffers are not cleared: each deflated pole and each
    solved eigenvalue has to be there once)."""
    kept = np.unique(pr.d[pr.z != 0.0])
    rows = np.sort(np.concatenate([pr.d[pr.z == 0.0]] + [
        np.full(c - 1, v) for v, c in zip(*np.unique(pr.d[pr.z != 0.0], return_counts=True))]))
    defl = (r["info"] & DEFLATED) != 0
    assert np.array_equal(np.sort(r["lam"][defl]), rows)
    assert np.count_nonzero(~defl) == kept.size + 1
    return defl


@pytest.mark.parametrize("name, pr", C.cases(), ids=[n for n, _ in C.cases()])
def test_columns(name, pr, finish, oracle_lib):
    for q in _widened(pr):
        r = emu.solve(0, q.d, q.z, q.scalar)
        defl = _once(q, r)
        assert np.all(r["lam"][:-1] >= r["lam"][1:])
        ks = np.arange(q.n) if q.n <= 150 else np.unique(np.concatenate(
            [np.arange(0, q.n, q.n // 30), np.nonzero(defl)[0][::8], np.nonzero(r["info"] & 6)[0][:30]]))
        ref = oracle.arrow_eig(q.d, q.z, q.scalar, ks=ks)
        assert_close(r["lam"][ks], ref.lam, name + " values")
        assert_close(r["V"][:, ks], ref.vec, name + " vectors")
        assert np.array_equal(defl[ks], ref.tau == 0)


@pytest.mark.parametrize("remedies, tau_nu", [(0, 100.0), (1, 1e300), (1, 1.0)])
def test_columns_of_unrepaired_values(remedies, tau_nu, finish):
    """Without repairs the values may be far off and out of order; no pair is lost."""
    for _, pr in C.cases():
        for q in _widened(pr):
            _once(q, emu.solve(0, q.d, q.z, q.scalar, remedies=remedies, tau_nu=tau_nu))
