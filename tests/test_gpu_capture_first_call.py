"""The first call on a handle, which allocates its workspace, inside a relaxed stream capture: every
replay gives the eager result, with eager calls on the same handle and other work in between."""
import ctypes

import numpy as np
import pytest

from paper_1302_7203_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [100, 512, 1500])
def test_first_call_in_a_capture(n):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    L = binding.lib()
    rng = np.random.default_rng(n)
    probs = [W.uniform_arrow(n, rng) for _ in range(3)]
    for q in probs[1:]:
        q.d, q.scalar = rng.permutation(q.d), probs[0].scalar   # the scalar is part of the captured call
    want = []
    for q in probs:
        out = binding.arrow_eig(torch.from_numpy(q.d).to(dev), torch.from_numpy(q.z).to(dev), q.scalar)
        want.append((out.lam.clone(), out.V.t().clone()))
    d, z = torch.from_numpy(probs[0].d).to(dev), torch.from_numpy(probs[0].z).to(dev)
    lam = torch.empty(n, dtype=torch.float64, device=dev)
    V = torch.empty((n, n), dtype=torch.float64, device=dev)
    h = ctypes.c_void_p()
    assert L.arrow_create(ctypes.byref(h), 0) == 0
    binding.apply_tuned(h)   # the lanes of the default handle, so the same bits

    def call():
        binding._bind_stream(h, dev)
        return L.arrow_eig(h, n, binding._ptr(d), binding._ptr(z), probs[0].scalar, binding._ptr(lam), binding._ptr(V),
                           n, None, None, None)

    torch.cuda.synchronize(dev)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        rc = call()
    assert rc == 0
    for turn in range(6):
        q = probs[turn % 3]
        d.copy_(torch.from_numpy(q.d))
        z.copy_(torch.from_numpy(q.z))
        lam.fill_(float("nan"))
        V.fill_(float("nan"))
        if turn % 2:
            assert call() == 0            # eager, on the captured call's workspace
            torch.cuda.synchronize(dev)
            assert torch.equal(lam, want[turn % 3][0])
        g.replay()
        torch.cuda.synchronize(dev)
        assert torch.equal(lam, want[turn % 3][0]) and torch.equal(V, want[turn % 3][1])
    del g
    assert L.arrow_destroy(h) == 0
