"""Kernels that took products from row groups, tiles and marches are no further from 64-bit sums than the order those take:
the entries of a row dealt to lanes in turn, a chain of multiply-adds on each, the chains added in pairs.  Both errors are measured on
the same operands, over the rows that have all their taps; the 2-norms of 10^5 and more results repeat to some 0.2 %, and
what one kernel's numbers do to the two orders is below 5 % (asserted: no larger; here they are 0.6 to 0.95 of it)."""
import numpy as np
import pytest
import torch

import paper_2411_19419_amd as cs
from gpu_util import device

pytestmark = pytest.mark.gpu


def _errors(storage, shape, batch, channels, lanes):
    """Relative 2-norm errors of conv_spmv and of the sums in `lanes` chains."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(91)
    K = rng.standard_normal((channels, k, k)).astype(np.float32)
    Kd = torch.from_numpy(K.reshape(-1)).to(device())
    if storage == "compact":
        plan = cs.conv_compact_build(*shape, Kd, channels=channels)
    elif channels > 1:
        plan = cs.conv_csr_build_channels(*shape, Kd, channels)
    else:
        plan = cs.conv_csr_build(*shape, Kd)
    x = rng.standard_normal((channels, m, n, batch)).astype(np.float32)
    y = cs.conv_spmv(plan, torch.from_numpy(x.reshape(-1)).to(device()), batch=batch).cpu().numpy()
    variant = plan.variant(batch)
    plan.close()
    inner = slice(-(-p // s), (m + p - k) // s + 1), slice(-(-p // s), (n + p - k) // s + 1)      # outputs with all taps
    y = y.reshape(plan.m_out, plan.n_out, batch)[inner]
    ax, ay = inner[0].start * s - p, inner[1].start * s - p
    taps = [(K[c, a, b], x[c, ax + a:ax + a + s * (y.shape[0] - 1) + 1:s, ay + b:ay + b + s * (y.shape[1] - 1) + 1:s])
            for c in range(channels) for a in range(k) for b in range(k)]
    exact = np.zeros(y.shape)
    chains = [np.zeros(y.shape, np.float32) for _ in range(lanes)]
    for t, (w, pixels) in enumerate(taps):
        exact += np.float64(w) * pixels
        chains[t % lanes] = (np.float64(w) * pixels + chains[t % lanes]).astype(np.float32)      # (fma: the product is exact)
    while len(chains) > 1:
        chains = [chains[2 * i] + chains[2 * i + 1] for i in range(len(chains) // 2)]
    size = np.linalg.norm(exact)
    return variant, np.linalg.norm(y - exact) / size, np.linalg.norm(chains[0] - exact) / size


@pytest.mark.parametrize("shape,batch,channels,lanes", [
    ((75, 113, 5, 1, 2), 88, 1, 8), ((145, 210, 6, 2, 3), 96, 1, 8), ((209, 179, 8, 3, 4), 136, 1, 16), ((70, 75, 7, 3, 3), 101, 1, 8),
    ((136, 149, 5, 3, 2), 150, 5, 8), ((30, 34, 11, 1, 10), 518, 3, 16), ((101, 103, 1, 1, 0), 60, 92, 16), ((135, 184, 1, 4, 0), 281, 2, 1),
])
def test_items(shape, batch, channels, lanes):
    variant, got, before = _errors("csr", shape, batch, channels, lanes)
    assert "_items" in variant, variant
    assert got <= before, (variant, got, before)


# launches of a few workgroups less than compute units, taken from the row groups: lanes of one column and of four to sixteen
@pytest.mark.parametrize("shape,batch,lanes", [
    ((328, 476, 9, 1, 4), 1, 16), ((434, 466, 7, 1, 3), 2, 8), ((630, 466, 7, 2, 0), 3, 8), ((202, 241, 7, 1, 3), 32, 8), ((460, 420, 7, 2, 3), 12, 16),
])
def test_rectangles_in_place_of_row_groups(shape, batch, lanes):
    variant, got, before = _errors("compact", shape, batch, 1, lanes)
    assert variant.startswith("compact_rect_"), variant
    assert got <= before, (variant, got, before)


@pytest.mark.parametrize("shape,batch,lanes", [
    ((69, 97, 5, 2, 4), 300, 8), ((105, 122, 7, 1, 0), 42, 8), ((85, 92, 4, 1, 2), 204, 4), ((360, 306, 8, 1, 7), 3, 8),
])
def test_lanes_over_descriptors(shape, batch, lanes):
    variant, got, before = _errors("compact", shape, batch, 1, lanes)
    assert variant.startswith("compact_gather_lanes_"), variant
    assert got <= before, (variant, got, before)
