"""Bisection forms each norm in the first pass: the check leaves no pass to an eigenvalue that
needs no remedy, so that it lists none of them."""
import numpy as np
import pytest

from emu import emu
from paper_1302_7203_amd import workloads as W

MAKE = {W.KIND_ARROW: W.uniform_arrow, W.KIND_DPR1: W.dpr1, W.KIND_SVD: W.svd_arrow, W.KIND_HERM: W.herm_arrow}
REMEDIES = 2 | 4 | 8 | 512   # Remark 2(a), 2(b), Remark 1, the DPR1 re-measure


@pytest.mark.parametrize("kind", list(MAKE))
def test_no_check_pass_without_a_remedy(kind):
    pr = MAKE[kind](120, np.random.default_rng(kind))
    rational = emu.solve(kind, pr.d, pr.z, pr.scalar)
    r = emu.solve(kind, pr.d, pr.z, pr.scalar, root=0)
    plain = (r["info"] & REMEDIES) == 0
    assert np.count_nonzero(plain) > 60
    order = np.arange(pr.n)
    assert np.all(r["cnt"][order[plain], 3:] == 0)
    # ... and its root stage counts the pass
    same = plain & (rational["info"] == r["info"])
    assert np.all(r["cnt"][same, 2] == rational["cnt"][same, 2] + 1)
