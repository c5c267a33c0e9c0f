"""Segments of the staged march where several blocks of batch columns share the XCDs: the rounds that a launch takes (host), and
the results of such launches against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

# (shape, batch, storage): T (0) and T^T (1); batches of whole and of partial blocks, 16 and 4 columns wide; one, two and three rounds
SHAPES = [((147, 201, 7, 1, 0), 184, 0), ((120, 150, 7, 1, 3), 180, 0), ((754, 1033, 11, 4, 5), 12, 0), ((206, 268, 11, 2, 5), 48, 1),
          ((205, 264, 6, 1, 3), 48, 1), ((233, 144, 7, 1, 0), 80, 0), ((250, 387, 7, 1, 0), 37, 0), ((221, 326, 6, 1, 3), 164, 0)]


@pytest.mark.parametrize("shape,batch,storage", SHAPES)
def test_rounds_of_segments(shape, batch, storage):
    d = cs.conv_dispatch_info(*shape, batch, storage)
    assert d.kernel == 9
    lines, columns = (shape[0], shape[1]) if storage else cs.conv_out_shape(*shape)
    strips, blocks, step = -(-columns // d.strip), -(-batch // (4 * d.columns_per_lane // 4)), d.lines_per_step

    def cost(seg):      # rounds of 32 workgroups per XCD, each as long as a segment and two steps
        cells = strips * -(-lines // seg)
        return -(-(-(-cells // 8) * blocks) // 32) * (seg + 2 * step)

    assert cost(d.segment) == min(cost(seg) for seg in range(step, lines + step, step))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,batch,storage", SHAPES)
def test_products_of_these_segments(shape, batch, storage):
    m, n, k, s, p = shape
    rng = np.random.default_rng(96)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = (cs.conv_csc_build if storage else cs.conv_csr_build)(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch).startswith("lds_march_staged"), plan.variant(batch)
    x = rng.standard_normal(plan.cols * batch).astype(np.float32)
    conv = oracle.conv_t if storage else oracle.conv
    ref, scale = conv(m, n, k, s, p, x, K, batch=batch, want_scale=True)
    got = cs.conv_spmv(plan, torch.from_numpy(x).to(device()), batch=batch).cpu().numpy()
    assert np.all(np.abs(got.astype(np.float64) - ref) <= REL_TOL * scale)
    plan.close()
