"""Products from row descriptors with a lane per row and chunk of columns: which products take them (host), and their results against
the oracle where the kernel has its edges."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device
from test_gpu_compact import _decoded_reference, _word

LANES = [
    # every number of taps of a line that is built, one column per lane and four; batches that chunks of four do not divide,
    # strides, borders wider than the kernel, a wave of a few rows' many chunks and one of many rows
    ((200, 301, 2, 1, 1), 3), ((90, 91, 2, 2, 3), 30), ((400, 410, 3, 1, 1), 3), ((8, 343, 3, 1, 4), 39), ((555, 50, 4, 1, 5), 3), ((8, 628, 4, 2, 5), 62),
    ((500, 410, 5, 2, 2), 3), ((10, 201, 5, 1, 6), 69), ((30, 835, 6, 1, 7), 3), ((153, 12, 6, 1, 7), 86), ((80, 713, 7, 1, 3), 3), ((580, 19, 7, 2, 8), 61),
    ((653, 674, 8, 2, 4), 3), ((8, 237, 8, 1, 9), 87), ((442, 375, 9, 2, 4), 3), ((248, 9, 9, 1, 10), 69), ((416, 502, 10, 2, 0), 3), ((12, 162, 10, 1, 11), 94),
    ((23, 836, 11, 1, 12), 3), ((168, 13, 11, 1, 12), 90), ((565, 306, 12, 2, 6), 3), ((411, 8, 12, 1, 13), 51), ((453, 418, 13, 2, 14), 3), ((652, 8, 13, 1, 14), 34),
]


@pytest.mark.parametrize("shape,batch", LANES)
def test_which_products_take_lanes(shape, batch):
    d = cs.conv_dispatch_info(*shape, batch, 2)
    rows, columns = oracle.out_shape(*shape), 4 if batch >= 4 else 1
    items = rows[0] * rows[1] * -(-batch // columns)
    assert (d.kernel, d.lanes_per_row, d.columns_per_lane, d.workgroups) == (10, 1, columns, -(-items // 256))


@pytest.mark.gpu
@pytest.mark.parametrize("shape,batch", LANES)
def test_lanes(shape, batch):
    m, n, k, s, p = shape
    rng = np.random.default_rng(96)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch) == "compact_gather_lanes_" + ("float4" if batch >= 4 else "scalar"), plan.variant(batch)
    # one value off the alignment of a vector
    x = torch.zeros(m * n * batch + 1, device=device())[1:]
    values = rng.standard_normal(m * n * batch).astype(np.float32)
    values[[0, m * n * batch // 2]] = np.inf, np.nan
    x.copy_(torch.from_numpy(values))
    ref, scale = oracle.conv(m, n, k, s, p, values, K, batch=batch, want_scale=True)
    got = cs.conv_spmv(plan, x, batch=batch).cpu().numpy()
    finite = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), finite) and finite.any()
    assert np.all(np.abs(got[finite].astype(np.float64) - ref[finite]) <= REL_TOL * scale[finite])
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape,batch", [((153, 12, 6, 1, 7), 86), ((80, 713, 7, 1, 3), 3), ((652, 8, 13, 1, 14), 34)])
def test_lanes_follow_edited_descriptors(shape, batch):
    """Rows emptied, shortened, and moved among rows that have all taps: the rectangle of each decides, not its place in the output."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(97)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch).startswith("compact_gather_lanes"), plan.variant(batch)
    desc, ktab = plan.row_desc.cpu().numpy().copy(), plan.ktab.cpu().numpy().copy()
    rows = len(desc)
    for row in range(3, rows, 97):
        which = row // 97 % 4
        if which == 0: desc[row] = (0, 0)
        elif which == 1: desc[row] = ((m - 2) * n + n - 2, _word(k - 2, 2, 0, 2))      # the last pixels, under a corner of the kernel
        elif which == 2: desc[row] = (0, _word(0, min(k, m), 0, min(k, n)))
        else: desc[row] = (n - 2, _word(k - 1, 1, 1, k - 1))                           # on over the end of a line
    plan.row_desc.copy_(torch.from_numpy(desc).to(device()))
    x = rng.standard_normal(m * n * batch).astype(np.float32)
    got = cs.conv_spmv(plan, torch.from_numpy(x).to(device()), batch=batch).cpu().numpy().astype(np.float64)
    ref, scale = _decoded_reference(shape, desc, ktab, x, batch)
    assert np.all(np.abs(got - ref) <= REL_TOL * scale)
    plan.close()
