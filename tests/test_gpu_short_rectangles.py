"""Rectangles over row descriptors whose launch has fewer workgroups than compute units: which products take them (host), and
their results against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device


@pytest.mark.parametrize("shape,batch,kernel", [
    # strips that do not divide the workgroups asked for: long segments march, short ones do not
    ((3239, 2417, 7, 2, 3), 4, 5), ((642, 952, 7, 2, 6), 76, 5), ((461, 628, 5, 2, 2), 49, 5), ((3225, 3031, 3, 2, 0), 20, 5),
    ((301, 271, 2, 2, 1), 178, 10), ((422, 529, 3, 2, 1), 11, 10),
    # the shortest segments: workgroups by the taps, strips not mostly empty
    ((571, 726, 7, 1, 3), 1, 5), ((202, 241, 7, 1, 3), 32, 5), ((497, 778, 9, 1, 0), 1, 5), ((95, 100, 7, 1, 3), 32, 10), ((200, 200, 7, 1, 3), 1, 10),
    ((334, 520, 5, 1, 4), 1, 10), ((366, 535, 3, 1, 0), 7, 10),
])
def test_which_products_march(shape, batch, kernel):
    assert cs.conv_dispatch_info(*shape, batch, 2).kernel == kernel


@pytest.mark.gpu
@pytest.mark.parametrize("shape,batch", [((497, 778, 9, 1, 0), 1), ((202, 241, 7, 1, 3), 32), ((181, 275, 7, 2, 3), 38), ((461, 628, 5, 2, 2), 49),
                                         ((251, 329, 5, 1, 2), 12), ((571, 726, 7, 1, 3), 1)])
def test_short_rectangles(shape, batch):
    m, n, k, s, p = shape
    rng = np.random.default_rng(95)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch).startswith("compact_rect"), plan.variant(batch)
    x = rng.standard_normal(m * n * batch).astype(np.float32)
    x[m * n * batch // 2] = np.inf
    ref, scale = oracle.conv(m, n, k, s, p, x, K, batch=batch, want_scale=True)
    got = cs.conv_spmv(plan, torch.from_numpy(x).to(device()), batch=batch).cpu().numpy()
    finite = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), finite) and not finite.all()
    assert np.all(np.abs(got[finite].astype(np.float64) - ref[finite]) <= REL_TOL * scale[finite])
    plan.close()
