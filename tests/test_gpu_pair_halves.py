"""shift and mu are optional one by one: either alone is the half of the pair that a call with
both returns, also where calls without them run another kernel (n > 4608)."""
import numpy as np
import pytest

from paper_1302_7203_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [W.KIND_ARROW, W.KIND_HERM])
@pytest.mark.parametrize("n", [900, 5900])
def test_halves_equal_the_pair(kind, n):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    h, L = binding.handle(0), binding.lib()
    binding._bind_stream(h, dev)
    rng = np.random.default_rng(n)
    pr = W.graded_arrow(n, rng)
    if kind == W.KIND_HERM:
        pr.z = pr.z * np.exp(1j * rng.uniform(0, 6.28, n - 1))
    d, z = torch.from_numpy(pr.d).to(dev), torch.from_numpy(pr.z).to(dev)
    f = L.arrow_eig_herm if kind == W.KIND_HERM else L.arrow_eig

    def solve(shift, mu):
        out = [torch.full((n,), float("nan"), dtype=torch.float64, device=dev) for _ in range(3)]
        assert f(h, n, binding._ptr(d), binding._ptr(z), pr.scalar, binding._ptr(out[0]), None, n,
                 binding._ptr(out[1]) if shift else None, binding._ptr(out[2]) if mu else None, None) == 0
        torch.cuda.synchronize(dev)
        return out

    lam, shift, mu = solve(True, True)
    assert not bool(mu.isnan().any())
    assert torch.equal(solve(True, False)[1], shift)
    alone = solve(False, True)
    assert torch.equal(alone[2], mu) and torch.equal(alone[0], lam)
