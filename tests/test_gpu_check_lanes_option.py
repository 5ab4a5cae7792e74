"""ARROW_OPT_CHECK_LANES stays accepted with the values it had, and changes nothing."""
import ctypes

import numpy as np
import pytest

from paper_1302_7203_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_accepted_without_effect():
    import torch
    from paper_1302_7203_amd import batch, binding
    rng = np.random.default_rng(8)
    probs = [W.uniform_arrow(90, rng), W.dpr1(33, rng), W.graded_arrow(200, rng)]
    results = []
    try:
        for lanes in (4, 0, 8, 16, 32, 64):
            binding.set_option(binding.OPT_CHECK_LANES, lanes)
            b = batch.Batch(probs, device=torch.device("cuda", 0))
            b.run()
            torch.cuda.synchronize()
            results.append((b.out_pool.clone(), b.info_pool.clone()))
            b.close()
        f, h = binding.lib().arrow_set_option, binding.handle(0)
        assert [f(h, binding.OPT_CHECK_LANES, ctypes.c_double(v)) for v in (1, 2, 5, 128, -4, 4.5)] == [-3] * 6
    finally:
        binding.set_option(binding.OPT_CHECK_LANES, 4)
    for out, info in results[1:]:
        assert torch.equal(out, results[0][0]) and torch.equal(info, results[0][1])
