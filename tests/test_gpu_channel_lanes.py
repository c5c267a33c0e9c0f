"""One-launch channel sum over row descriptors with lanes of four columns: small planes whose last tiles are partly empty, kernel
sizes with unrolled taps and others, as built and with edited descriptors; chunks side by side where the dispatch has them
(every such kernel by name: test_gpu_channel_parts.py).  Reference: the sliding-window oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,channels,batch", [
    ((9, 17, 3, 1, 1), 20, 16), ((6, 4, 1, 1, 0), 33, 32), ((5, 13, 7, 2, 3), 9, 16), ((11, 30, 5, 1, 2), 4, 48), ((21, 9, 3, 2, 1), 64, 8),
    ((8, 23, 2, 1, 1), 17, 24), ((13, 12, 11, 1, 5), 6, 16), ((20, 19, 9, 3, 4), 5, 40), ((7, 18, 4, 1, 3), 12, 12),
])
def test_chunks_side_by_side(shape, channels, batch):
    m, n, k, s, p = shape
    rng = np.random.default_rng(81)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()), channels=channels)
    assert plan.variant(batch).startswith("compact_channels_4x16_float4x1"), plan.variant(batch)
    x = rng.standard_normal(plan.cols * batch).astype(np.float32)
    xd = torch.from_numpy(x).to(device())
    ref, scale = oracle.conv_channels(m, n, k, s, p, x, K, channels, batch=batch, want_scale=True)
    y = torch.full((plan.rows * batch,), float("nan"), device=device())
    cs.conv_spmv(plan, xd, y, batch=batch)
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref.astype(np.float64)) <= REL_TOL * scale)
    # a row emptied: its outputs are zero, the others as before
    row = plan.rows // 2
    desc = plan.row_desc.cpu().numpy().copy()
    desc[row] = 0
    plan.row_desc.copy_(torch.from_numpy(desc))
    got = cs.conv_spmv(plan, xd, batch=batch).cpu().numpy().reshape(-1, batch).astype(np.float64)
    want, bound = ref.reshape(-1, batch).astype(np.float64), scale.reshape(-1, batch).copy()
    want[row] = 0.0
    assert np.array_equal(got[row], want[row]) and np.all(np.abs(got - want) <= REL_TOL * bound)
    plan.close()
