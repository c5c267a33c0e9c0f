"""Where items and descriptor lanes take products from the other kernels, against the times that the lines were drawn over
(profiles/chunk_kernel_times.csv): queried on the host, no GPU."""
import csv
import math
import os

import pytest

import paper_2411_19419_amd as cs

TIMES = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "profiles", "chunk_kernel_times.csv")
STORAGE = {"csr": 0, "csc": 1, "compact": 2}


def _rows():
    with open(TIMES) as f:
        for r in csv.DictReader(f):
            shape = tuple(int(r[x]) for x in "mnksp")
            d = cs.conv_dispatch_info(*shape, int(r["batch"]), STORAGE[r["storage"]], int(r["channels"]))
            yield r, math.log(float(r["other_us"]) / float(r["chunks_us"])), d.strip > 0 and d.kernel in (0, 1, 10)


# products timed, slower ones among those taken (share), and the mean gain over all as a share of the best choice's
@pytest.mark.parametrize("which,slower,share", [("items", 0.04, 0.9), ("items of two or three columns", 0.015, 0.95), ("lanes", 0.01, 0.60)])
def test_products_taken_are_the_faster_ones(which, slower, share):
    rows = [r for r in _rows() if (r[0]["storage"] == "compact") == (which == "lanes") and r[0]["held"] == "0"]
    if which.endswith("columns"):
        rows = [r for r in rows if r[0]["batch"] in "23" and r[0]["channels"] == "1"]
    assert len(rows) >= 1200
    taken = [gain for _, gain, takes in rows if takes]
    assert len(taken) >= 700 and sum(gain < -0.06 for gain in taken) <= slower * len(taken)
    assert sum(taken) >= share * sum(max(gain, 0.0) for _, gain, _ in rows)


def test_held_products_stay_where_they_are():
    for r, _, takes in _rows():
        if r["held"] != "0":
            assert takes == (int(r["held"]) > 0), r


# beyond the ranges of those products: batches and channels like the largest timed
@pytest.mark.parametrize("shape,batch,storage,channels", [((100, 100, 6, 3, 3), 16000, 0, 1), ((90, 91, 6, 3, 5), 40000, 0, 1), ((64, 64, 3, 1, 1), 5000, 1, 1),
                                                          ((50, 50, 5, 2, 2), 64, 0, 8000), ((40, 40, 3, 2, 1), 30000, 2, 1)])
def test_beyond_the_times(shape, batch, storage, channels):
    d = cs.conv_dispatch_info(*shape, batch, storage, channels)
    near = cs.conv_dispatch_info(*shape, min(batch, 2048), storage, min(channels, 1024))
    assert d.workgroups > 0 and (d.strip > 0, d.kernel) == (near.strip > 0, near.kernel)


# batches that fill the lanes of the kernels left (2 or 4 chunks each), where those are at their best; products of T, of T^T and channel
# sums apart, as one may be wrong while the others hide it
def test_batches_that_fill_the_other_kernels_lanes():
    groups = {}
    for r, gain, takes in _rows():
        chunks = int(r["other_chunks_per_lane"])
        if r["storage"] != "compact" and r["held"] == "0" and chunks > 1 and int(r["batch"]) % (4 * chunks) == 0 and takes:
            groups.setdefault((r["storage"], r["channels"] == "1"), []).append(gain)
    assert len(groups) == 3
    for group, taken in groups.items():
        assert len(taken) >= 100 and sum(gain < -0.06 for gain in taken) <= 0.06 * len(taken), (group, len(taken), sum(gain < -0.06 for gain in taken))
