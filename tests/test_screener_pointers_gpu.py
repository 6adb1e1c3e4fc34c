"""A training step takes rows and targets as device addresses too, as the single calls do."""
import numpy as np
import pytest

from paper_2412_00802_amd.screener import D_IN, Screener, init_params

pytestmark = pytest.mark.gpu


def test_training_step_takes_addresses():
    import torch
    rng = np.random.default_rng(2)
    x = torch.from_numpy((rng.random((64, D_IN)) < 0.004).astype(np.float32)).cuda().bfloat16()
    y = torch.from_numpy(rng.random((64, 2)).astype(np.float32)).cuda()
    a, b = (Screener(init_params(seed=5), batch=64) for _ in range(2))
    a.train_step(64, y, x)
    b.train_step(64, y.data_ptr(), x.data_ptr())
    for k in a.p:
        assert torch.equal(a.p[k], b.p[k]), k
