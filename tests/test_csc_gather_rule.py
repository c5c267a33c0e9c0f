"""Host logic of the gathering product from the column-compressed arrays (no GPU needed): what its kernel
assumes of the strip, the segments and its LDS, and which shapes it leaves to the scatter."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2411_19419_amd import binding


def gather_info(m, n, k, s, p, batch, jobs=256):
    d = binding.ConvDispatch()
    st = binding._load().conv_test_csc_gather_info(m, n, k, s, p, batch, jobs, ctypes.byref(d))
    assert st == 0, (st, m, n, k, s, p, batch)
    return {name: getattr(d, name) for name, _ in d._fields_}


def test_geometry_over_many_shapes():
    rng = np.random.default_rng(17)
    seen = 0
    for _ in range(600):
        k, s, p = int(rng.integers(1, 16)), int(rng.integers(1, 6)), int(rng.integers(0, 14))
        m, n = (int(v) for v in rng.integers(max(1, k - 2 * p), 2500, size=2))
        if oracle.nnz_closed(m, n, k, s, p) >= 2 ** 31:
            continue
        mo, no = oracle.out_shape(m, n, k, s, p)
        kl = -(-k // s)
        for batch in (1, 3, 4, 5, 9, 16, 17, 64):
            d = gather_info(m, n, k, s, p, batch, jobs=1)
            if d["kernel"] == 0:
                continue
            seen += 1
            assert s <= k and p < k and kl <= 13
            lanes, cols, tw, ways = d["lanes_per_row"], d["columns_per_lane"], d["strip"], d["lines_per_step"]
            assert cols == (1 if batch < 4 else 4) and lanes == (1 if batch <= 4 else 2 if batch <= 8 else 4)
            assert tw in (16, 32, 64) and tw * lanes * ways == d["threads"] == 256     # every lane has a share of one output column
            assert d["lds_bytes"] <= 64 * 1024 and d["ring_lines_needed"] == kl
            # five accesses per thread and array hold the longest line: the windows over the strip's pixels, kl lines of them
            covered = [sum(1 for w in range((j + p) // s + 1) if j + p - s * w < k and w < no) for j in range(min(n, (tw - 1) * s + k))]
            assert sum(covered) * kl <= 4 * d["ring_lines"] <= 4 * 5 * 256
            strips, segs = -(-no // tw), -(-mo // d["segment"])
            assert d["workgroups"] == strips * segs * -(-batch // (cols * lanes)) < 2 ** 18
    assert seen > 1000


@pytest.mark.parametrize("shape,batch,gathers", [
    ((1024, 1024, 7, 1, 3), 16, True), ((1024, 1024, 7, 1, 3), 1, True), ((4096, 4096, 11, 4, 5), 4, True),
    # little work for a line's fixed cost
    ((32, 40, 7, 1, 3), 16, False), ((137, 210, 11, 1, 5), 1, False), ((691, 628, 13, 2, 0), 3, False), ((176, 128, 7, 1, 3), 8, False),
    ((92, 79, 7, 1, 3), 48, False), ((564, 447, 8, 1, 4), 3, False), ((241, 336, 7, 1, 0), 2, False), ((183, 123, 8, 1, 0), 16, False),
    ((1292, 1151, 1, 1, 0), 4, False), ((1292, 1151, 1, 1, 0), 5, True), ((427, 533, 3, 2, 1), 1, False), ((427, 533, 4, 2, 1), 1, True),
    ((3384, 3491, 1, 1, 0), 1, False), ((1226, 786, 2, 1, 0), 1, False),       # an entry or four per pixel, one vector
    ((1000, 1000, 3, 4, 1), 16, False), ((1000, 1000, 5, 1, 5), 16, False),    # pixels, rows without entries
    ((1000, 1000, 14, 1, 7), 16, False), ((5, 1, 5, 1, 4), 4, False),
])
def test_which_shapes_gather(shape, batch, gathers):
    info = gather_info(*shape, batch)
    assert info["kernel"] == (11 if gathers else 0)
    # the public report is that of the kernel that runs
    d = binding.conv_dispatch_info(*shape, batch, 3)
    assert (d.kernel == 11) == gathers and (gathers or d.kernel in (7, 8))
    assert not gathers or info == {name: getattr(d, name) for name, _ in d._fields_}


def test_argument_checks():
    lib, d = binding._load(), binding.ConvDispatch()
    assert lib.conv_test_csc_gather_info(8, 8, 3, 1, 1, 4, 1, None) == -2
    assert lib.conv_test_csc_gather_info(8, 8, 3, 1, 1, 0, 1, ctypes.byref(d)) == -1
    assert lib.conv_test_csc_gather_info(8, 8, 11, 1, 1, 4, 1, ctypes.byref(d)) == -1
    assert lib.conv_test_csc_gather_info(40000, 40000, 3, 1, 1, 4, 1, ctypes.byref(d)) == -3
