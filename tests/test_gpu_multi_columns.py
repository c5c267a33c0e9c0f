"""Many products in one launch: a lane's batch columns, one to three by themselves and from four on in chunks, against the
single products and the oracle; rows shorter and longer than a lane's entries asked for together."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

pytestmark = pytest.mark.gpu

SHAPES = [(7, 9, 1, 1, 0), (16, 15, 3, 1, 1), (9, 30, 3, 2, 4), (20, 21, 7, 2, 3), (12, 13, 2, 2, 0), (17, 11, 11, 1, 5), (14, 14, 5, 3, 2)]


@pytest.mark.parametrize("batch", [1, 2, 3, 4, 5, 7, 8, 9, 13, 16, 17])
def test_columns_of_many_products(batch):
    rng = np.random.default_rng(91)
    Ks = [rng.standard_normal(k * k).astype(np.float32) for _, _, k, _, _ in SHAPES]
    xs = [rng.standard_normal(m * n * batch).astype(np.float32) for m, n, *_ in SHAPES]
    plans = [cs.conv_csr_build(*shape, torch.from_numpy(K).to(device())) for shape, K in zip(SHAPES, Ks)]
    ys = [torch.full((plan.rows * batch + 8,), float("nan"), device=device())[1:1 + plan.rows * batch] for plan in plans]
    multi = cs.ConvMulti(plans, [torch.from_numpy(x).to(device()) for x in xs], ys, batch=batch)
    multi.apply()
    torch.cuda.synchronize()
    for shape, K, x, y in zip(SHAPES, Ks, xs, ys):
        ref, scale = oracle.conv(*shape, x, K, batch=batch, want_scale=True)
        assert np.all(np.abs(y.cpu().numpy().astype(np.float64) - ref.astype(np.float64)) <= REL_TOL * scale), (shape, batch)
    multi.close()
    for plan in plans:
        plan.close()
