"""One-launch channel sum over row descriptors with tiles in parts, chunks of batch columns side by side: where the dispatch takes how
many (host), and the results of every compiled combination against the oracle, as built and with an edited descriptor."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

# shape, channels, batch, chunks side by side
PARTS = [
    # pixels in flight per lane: 4, 8; unrolled taps (k 1 and 3) and any; the last tiles with outputs in some of their parts
    ((26, 43, 1, 1, 0), 33, 16, 4), ((27, 31, 1, 3, 0), 9, 32, 4), ((29, 35, 3, 1, 1), 20, 16, 4), ((31, 50, 3, 2, 1), 11, 16, 4), ((13, 21, 5, 1, 2), 6, 16, 4),
    ((17, 38, 6, 2, 1), 3, 16, 2), ((15, 34, 4, 3, 3), 12, 16, 1), ((25, 39, 1, 2, 0), 40, 24, 2), ((40, 44, 1, 3, 0), 5, 8, 2), ((25, 35, 3, 1, 0), 17, 24, 2),
    ((33, 52, 3, 2, 2), 64, 24, 2), ((12, 19, 6, 1, 3), 14, 16, 2), ((20, 33, 9, 1, 4), 7, 40, 2), ((21, 19, 5, 2, 2), 5, 24, 2), ((18, 23, 2, 2, 1), 16, 16, 4),
    # ragged batches, overlaps that would need more pixels in flight, few workgroups of k 3 (enough at stride 2):
    # one chunk
    ((26, 43, 1, 1, 0), 33, 12, 1), ((26, 19, 7, 1, 0), 3, 16, 1), ((35, 42, 6, 1, 0), 4, 16, 2), ((90, 62, 8, 1, 0), 19, 8, 1), ((30, 28, 3, 1, 1), 47, 8, 1),
    ((18, 17, 3, 2, 1), 163, 16, 1), ((19, 29, 3, 2, 1), 113, 32, 4), ((16, 19, 3, 3, 1), 41, 16, 1),
]


@pytest.mark.parametrize("shape,channels,batch,chunks", PARTS)
def test_chunks_side_by_side(shape, channels, batch, chunks):
    d = cs.conv_dispatch_info(*shape, batch, 2, channels)
    assert (d.kernel, d.columns_per_lane, d.strip) == (6, 4, 16 // chunks)
    mo, no = cs.conv_out_shape(*shape)
    assert d.workgroups == -(-mo // 4) * -(-no // 16) * (batch // 4)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,channels,batch,chunks", PARTS)
def test_results(shape, channels, batch, chunks):
    m, n, k, s, p = shape
    rng = np.random.default_rng(83)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()), channels=channels)
    x = rng.standard_normal(plan.cols * batch).astype(np.float32)
    xd = torch.from_numpy(x).to(device())
    ref, scale = oracle.conv_channels(m, n, k, s, p, x, K, channels, batch=batch, want_scale=True)
    want, bound = ref.reshape(-1, batch).astype(np.float64), scale.reshape(-1, batch)
    for edited in (False, True):
        if edited:      # a row emptied: its outputs are zero, the others as before
            desc = plan.row_desc.cpu().numpy().copy()
            desc[plan.rows // 3] = 0
            plan.row_desc.copy_(torch.from_numpy(desc))
            want[plan.rows // 3] = 0.0
        y = torch.full((plan.rows * batch,), float("nan"), device=device())
        got = cs.conv_spmv(plan, xd, y, batch=batch).cpu().numpy().reshape(-1, batch).astype(np.float64)
        assert np.all(np.abs(got - want) <= REL_TOL * bound), (shape, edited)
    plan.close()
