"""A lanes table that the caller sets holds at every order; the measured default table leaves
orders above 4608 to the large problems' kernel."""
import numpy as np
import pytest

from paper_1302_7203_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [W.KIND_ARROW, W.KIND_DPR1])
def test_callers_table_above_4608(kind):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(2)
    pr = (W.uniform_arrow if kind == W.KIND_ARROW else W.dpr1)(6000, rng)
    d, z = torch.from_numpy(pr.d).to(dev), torch.from_numpy(pr.z).to(dev)
    h = binding.handle(0)
    f = binding.arrow_eig if kind == W.KIND_ARROW else binding.dpr1_eig

    def solve(table=None, option=0):
        if table:
            binding.set_lanes_table(binding.SCHEDULE_SINGLE, [binding.INT32_MAX], [table], h=h)
        binding.set_option(binding.OPT_LANES, option)
        try:
            out = f(d, z, pr.scalar, vectors=False)
            torch.cuda.synchronize(dev)
        finally:
            binding.set_option(binding.OPT_LANES, 0)
            if table:
                binding.apply_tuned(h)
        return out.lam

    fixed = {g: solve(option=g) for g in (8, 64)}
    assert not torch.equal(fixed[8], fixed[64])          # sums over other lanes: other last bits
    assert torch.equal(solve(table=8), fixed[8])
    assert torch.equal(solve(table=64), fixed[64])       # the large problems' kernel sums as 64 lanes do
    assert torch.equal(solve(), fixed[64])               # the default table (32 lanes here) does not reach it
    assert torch.equal(solve(table=64, option=8), fixed[8])
