"""Segments of marches over row descriptors where several blocks of batch columns share the XCDs: one round instead of a second one
for a few workgroups (host), and results against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

# longer segments and shorter ones; whole and partial blocks of columns; every compiled kernel of stride 2 that has its unit alone
SHAPES = [((165, 165, 7, 2, 3), 96), ((252, 342, 7, 2, 6), 80), ((279, 276, 5, 2, 2), 184), ((536, 333, 3, 2, 1), 184), ((338, 369, 5, 2, 4), 184),
          ((555, 789, 7, 2, 3), 37)]


@pytest.mark.parametrize("shape,batch", SHAPES)
def test_workgroups_fill_whole_rounds(shape, batch):
    d = cs.conv_dispatch_info(*shape, batch, 2)
    assert d.kernel == 5 and d.segment % d.lines_per_step == 0
    lines, columns = cs.conv_out_shape(*shape)
    cells = -(-columns // d.strip) * -(-lines // d.segment)
    blocks = d.workgroups // cells
    share = -(-cells // 8) * blocks
    assert share / 32 > 0.7 * -(-share // 32)       # the last round of 32 workgroups per XCD is not nearly empty


@pytest.mark.gpu
@pytest.mark.parametrize("shape,batch", SHAPES)
def test_products_of_these_segments(shape, batch):
    m, n, k, s, p = shape
    rng = np.random.default_rng(97)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch).startswith("compact_rect"), plan.variant(batch)
    x = rng.standard_normal(m * n * batch).astype(np.float32)
    ref, scale = oracle.conv(m, n, k, s, p, x, K, batch=batch, want_scale=True)
    got = cs.conv_spmv(plan, torch.from_numpy(x).to(device()), batch=batch).cpu().numpy()
    assert np.all(np.abs(got.astype(np.float64) - ref) <= REL_TOL * scale)
    plan.close()
