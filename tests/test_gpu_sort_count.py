"""The sort's count of finished blocks lies in the workspace between calls.  A value that calls
overlapping in one workspace left there must not outlive the next ordered call."""
import ctypes

import numpy as np
import pytest

from paper_1302_7203_amd import workloads as W

pytestmark = pytest.mark.gpu

COUNT = 7 * 8   # of the workspace's header, in bytes


def _handle(binding):
    h = ctypes.c_void_p()
    assert binding.lib().arrow_create(ctypes.byref(h), 0) == 0
    return h


def _solve(binding, h, pr, dev):
    import torch
    d, z = torch.from_numpy(pr.d).to(dev), torch.from_numpy(pr.z).to(dev)
    lam = torch.full((pr.n,), float("nan"), dtype=torch.float64, device=dev)
    binding._bind_stream(h, dev)
    assert binding.lib().arrow_eig(h, pr.n, binding._ptr(d), binding._ptr(z), pr.scalar, binding._ptr(lam), None, pr.n,
                                   None, None, None) == 0
    torch.cuda.synchronize(dev)
    return lam


@pytest.mark.parametrize("left", [1, 3, 200])
@pytest.mark.parametrize("n", [500, 1400])   # both launches that finish a call; several blocks sort
def test_next_call_starts_from_zero(n, left):
    import torch
    from paper_1302_7203_amd import binding
    dev = torch.device("cuda", 0)
    L = binding.lib()
    rng = np.random.default_rng(n)
    first, other = W.uniform_arrow(n, rng), W.uniform_arrow(n, rng)
    other.d, other.scalar = 100.0 * rng.permutation(other.d), 7.0
    h, ref = _handle(binding), _handle(binding)
    want = _solve(binding, h, first, dev), _solve(binding, ref, other, dev)
    ws = ctypes.c_uint64.from_address(h.value + 16).value   # the handle: device, stream, workspace
    word = ctypes.c_uint32(left)
    L.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]

    def copy(dst, src, kind):
        assert L.hipMemcpy(dst, src, 4, kind) == 0

    copy(ws + COUNT, ctypes.addressof(word), 1)
    # the same problem again: its workspace holds the same entries, whichever block reduces them
    assert torch.equal(_solve(binding, h, first, dev), want[0])
    copy(ctypes.addressof(word), ws + COUNT, 2)
    assert word.value == 0
    assert torch.equal(_solve(binding, h, other, dev), want[1])
    for x in (h, ref):
        assert L.arrow_destroy(x) == 0
