"""Batches that are not a multiple of 4 and operands that start anywhere, through every kernel of
the CSR and CSC storages: the last chunk of four columns starts at batch - 4, so columns are
computed by two lanes, and 16-byte accesses start at any float.  Reference: the sliding-window
oracle; the floats around the result must stay as they were."""
import numpy as np
import pytest
import scipy.sparse
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device, keep_to_the_scatter

pytestmark = pytest.mark.gpu


def _padded(a, offset):
    buf = torch.full((a.size + 8,), 7.0, dtype=torch.float32, device=device())
    buf[offset:offset + a.size] = torch.from_numpy(a).to(device())
    return buf, buf[offset:offset + a.size]


def _check(got, ref, scale, what):
    err = np.abs(got.astype(np.float64) - ref.astype(np.float64))
    assert not np.any(np.isnan(got)), what
    assert np.all(err <= REL_TOL * scale), what


KINDS = [   # shape, test threshold for the marching kernels (None: the default), what takes it
    ((64, 90, 3, 1, 1), None, "block_"), ((260, 200, 3, 1, 1), None, "lds_tile_"), ((120, 101, 5, 2, 2), None, "lds_tile_"), ((20, 33, 4, 1, 2), None, "gather_"),
    ((70, 75, 5, 1, 2), 1, "lds_march_staged_"), ((40, 75, 9, 1, 4), 1, "lds_march_staged_"),
    ((40, 75, 11, 1, 5), 1, "lds_march_staged_"), ((70, 131, 5, 2, 2), 1, "lds_march_"), ((70, 67, 10, 2, 3), 1, "lds_march_"),
]


@pytest.mark.parametrize("shape,jobs,kind", KINDS)
def test_ragged_batches_and_unaligned_operands(shape, jobs, kind):
    m, n, k, s, p = shape
    rng = np.random.default_rng(17)
    K = rng.standard_normal(k * k).astype(np.float32)
    Kd = torch.from_numpy(K).to(device())
    plan, plan_t = cs.conv_csr_build(*shape, Kd), cs.conv_csc_build(*shape, Kd)
    if jobs:
        for pl in (plan, plan_t):
            cs.conv_plan_set_march_min_jobs(pl, jobs)
    seen = set()
    for i, batch in enumerate((2, 3, 4, 5, 7, 8, 9, 10, 13, 16, 17, 22, 31, 100, 131)):
        offset = i % 4
        seen.add(plan.variant(batch).startswith(kind))
        x = rng.standard_normal(m * n * batch).astype(np.float32)
        y0 = np.full(plan.rows * batch, np.nan, dtype=np.float32)
        (_, xd), (yb, yd) = _padded(x, offset), _padded(y0, 3 - offset)
        cs.conv_spmv(plan, xd, yd, batch=batch)
        u = rng.standard_normal(plan.rows * batch).astype(np.float32)
        z0 = np.full(m * n * batch, np.nan, dtype=np.float32)
        (_, ud), (zb, zd) = _padded(u, offset), _padded(z0, 3 - offset)
        cs.conv_spmv(plan_t, ud, zd, batch=batch)
        torch.cuda.synchronize()
        _check(yd.cpu().numpy(), *oracle.conv(m, n, k, s, p, x, K, batch=batch, want_scale=True), (shape, batch))
        _check(zd.cpu().numpy(), *oracle.conv_t(m, n, k, s, p, u, K, batch=batch, want_scale=True), (shape, batch, "T"))
        for buf, size in ((yb, y0.size), (zb, z0.size)):
            edge = buf.cpu().numpy()
            assert np.all(edge[:3 - offset] == 7.0) and np.all(edge[3 - offset + size:] == 7.0)
    assert True in seen                       # the kernel this row is about ran for some of the batches
    plan.close()
    plan_t.close()


TILES = [   # T or T^T, batches: enough multiply-adds for the tile kernel
    ("csr", (260, 200, 3, 1, 1), (8, 9, 10, 13, 16, 31)), ("csr", (240, 251, 5, 2, 2), (10, 13, 16)),
    ("csc", (500, 450, 3, 1, 1), (6, 7, 9, 10, 13, 16)), ("csc", (500, 451, 5, 2, 2), (9, 10, 13, 16)),
]


@pytest.mark.parametrize("storage,shape,batches", TILES)
def test_tiles_at_ragged_batches(storage, shape, batches):
    m, n, k, s, p = shape
    rng = np.random.default_rng(41)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = (cs.conv_csr_build if storage == "csr" else cs.conv_csc_build)(*shape, torch.from_numpy(K).to(device()))
    for i, batch in enumerate(batches):
        offset = i % 4
        assert plan.variant(batch).startswith("lds_tile_"), (batch, plan.variant(batch))
        x = rng.standard_normal(plan.cols * batch).astype(np.float32)
        y0 = np.full(plan.rows * batch, np.nan, dtype=np.float32)
        (_, xd), (yb, yd) = _padded(x, offset), _padded(y0, 3 - offset)
        cs.conv_spmv(plan, xd, yd, batch=batch)
        torch.cuda.synchronize()
        _check(yd.cpu().numpy(), *(oracle.conv if storage == "csr" else oracle.conv_t)(m, n, k, s, p, x, K, batch=batch, want_scale=True),
               (shape, batch))
        edge = yb.cpu().numpy()
        assert np.all(edge[:3 - offset] == 7.0) and np.all(edge[3 - offset + y0.size:] == 7.0)
    plan.close()


@pytest.mark.parametrize("storage,shape,batches", TILES)
def test_tiles_read_the_stored_columns(storage, shape, batches):
    """Columns redirected after the build (far from the row's window, one pixel beside it, another
    line): the product follows the stored arrays, and no other row changes."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(43)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = (cs.conv_csr_build if storage == "csr" else cs.conv_csc_build)(*shape, torch.from_numpy(K).to(device()))
    rp, ci, va = oracle.csr(*shape, K)
    outputs = plan.m_out * plan.n_out
    T = scipy.sparse.csr_matrix((va.astype(np.float64), ci, rp), shape=(outputs, m * n))
    if storage == "csc":
        T = T.T.tocsr()
        T.sort_indices()
    ptr, idx = T.indptr, T.indices.copy()
    stored = plan.col_idx                      # (of a T^T plan: T's row numbers)
    assert np.array_equal(stored.cpu().numpy(), idx)
    rows = rng.choice(plan.rows, size=60, replace=False)
    rows = rows[np.diff(ptr)[rows] > 3]
    for i, row in enumerate(rows):
        e = ptr[row] + i % 4
        idx[e] = (0, plan.cols - 1, min(idx[e] + 1, plan.cols - 1), (idx[e] + 5 * n) % plan.cols)[i % 4]
    for batch in batches:
        assert plan.variant(batch).startswith("lds_tile_"), (batch, plan.variant(batch))
        x = rng.standard_normal(plan.cols * batch).astype(np.float32)
        xd = torch.from_numpy(x).to(device())
        stored.copy_(torch.from_numpy(T.indices))
        before = cs.conv_spmv(plan, xd, batch=batch).clone()
        stored.copy_(torch.from_numpy(idx))
        got = cs.conv_spmv(plan, xd, batch=batch)
        torch.cuda.synchronize()
        before, got = before.cpu().numpy().reshape(-1, batch), got.cpu().numpy().reshape(-1, batch)
        others = np.ones(plan.rows, bool)
        others[rows] = False
        assert np.array_equal(before[others], got[others])
        E = scipy.sparse.csr_matrix((T.data, idx, ptr), shape=T.shape)[rows]
        X = x.reshape(-1, batch).astype(np.float64)
        _check(got[rows], E @ X, abs(E) @ np.abs(X), (shape, batch))
    plan.close()


@pytest.mark.parametrize("shape", [(70, 75, 5, 1, 2), (70, 131, 5, 2, 2)])     # in one launch; a launch per channel, adding
@pytest.mark.parametrize("batch", [2, 5, 10, 19])
def test_ragged_batches_of_channel_sums(shape, batch):
    m, n, k, s, p = shape
    channels = 3
    rng = np.random.default_rng(batch)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    x = rng.standard_normal(channels * m * n * batch).astype(np.float32)
    plan = cs.conv_csr_build_channels(*shape, torch.from_numpy(K).to(device()), channels)
    cs.conv_plan_set_march_min_jobs(plan, 1)
    assert plan.variant(batch).startswith("lds_march_")
    y = cs.conv_spmv(plan, torch.from_numpy(x).to(device()), batch=batch)
    torch.cuda.synchronize()
    ref, scale = np.zeros(plan.rows * batch), np.zeros(plan.rows * batch)
    for c in range(channels):
        r, sc = oracle.conv(m, n, k, s, p, x[c * m * n * batch:(c + 1) * m * n * batch], K[c * k * k:(c + 1) * k * k],
                            batch=batch, want_scale=True)
        ref, scale = ref + r, scale + sc
    _check(y.cpu().numpy(), ref, scale, (shape, batch))
    plan.close()


def _row_group_error(w, lanes=16, samples=4000):
    """2-norm error of float32 sums of products with the numbers w in the row groups' order: `lanes`
    chains of fused multiply-adds over one list of all channels' entries, then a tree."""
    rng = np.random.default_rng(1)
    x = rng.standard_normal((w.size, samples)).astype(np.float32)
    parts = [np.zeros(samples, np.float32) for _ in range(lanes)]
    for t in range(w.size):           # (one rounding per step: the product is exact in 64 bits)
        parts[t % lanes] = (np.float64(w[t]) * x[t] + parts[t % lanes]).astype(np.float32)
    while len(parts) > 1:
        parts = [a + b for a, b in zip(parts[::2], parts[1::2])]
    ref = w.astype(np.float64) @ x
    return np.linalg.norm(parts[0] - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("shape,channels,batch,offset", [
    ((70, 75, 5, 1, 2), 64, 10, 0), ((70, 75, 7, 1, 3), 48, 5, 1), ((70, 75, 7, 1, 3), 3, 3, 0), ((70, 67, 7, 1, 3), 24, 8, 2),
    ((40, 75, 9, 1, 4), 24, 3, 0), ((130, 160, 11, 4, 5), 12, 5, 0),
])
def test_ragged_channel_sums_are_as_exact_as_the_row_groups(shape, channels, batch, offset):
    """Batches that are not a multiple of 4, or operands off the 16-byte grid, walked by the staged
    march: within 5 % (the scatter of the two samples) of the error of up to 16 lanes per row, where a
    single chain per lane through all channels is twice as far from the exact sum or more."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(channels)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    x = rng.standard_normal(channels * m * n * batch).astype(np.float32)
    plan = cs.conv_csr_build_channels(*shape, torch.from_numpy(K).to(device()), channels)
    cs.conv_plan_set_march_min_jobs(plan, 1)
    variant = plan.variant(batch)
    assert variant.startswith("lds_march_staged_") and variant.endswith("_%d_channels" % channels), variant
    _, xd = _padded(x, offset)
    y = cs.conv_spmv(plan, xd, batch=batch)
    torch.cuda.synchronize()
    ref, scale = oracle.conv_channels(m, n, k, s, p, x, K, channels, batch=batch, want_scale=True)
    got = y.cpu().numpy()
    _check(got, ref, scale, (shape, batch))
    ref = ref.astype(np.float64)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1.05 * _row_group_error(K)
    plan.close()


@pytest.mark.parametrize("shape,jobs,kind", [
    ((70, 75, 3, 1, 1), 1, "compact_rect"), ((60, 131, 5, 2, 2), 1, "compact_rect"), ((50, 75, 11, 1, 5), 1, "compact_described"),
    ((70, 75, 6, 4, 2), 1, "compact_described"), ((33, 41, 3, 1, 1), None, "compact_gather"), ((33, 41, 13, 1, 6), None, "compact_gather"),
])
def test_ragged_batches_from_the_structure_aware_storage(shape, jobs, kind):
    m, n, k, s, p = shape
    rng = np.random.default_rng(23)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()))
    if jobs:
        cs.conv_plan_set_march_min_jobs(plan, jobs)
    for i, batch in enumerate((2, 3, 4, 5, 7, 8, 9, 12, 13, 16, 18, 31, 57)):
        offset = i % 4
        assert plan.variant(batch).startswith(kind), plan.variant(batch)
        x = rng.standard_normal(m * n * batch).astype(np.float32)
        y0 = np.full(plan.rows * batch, np.nan, dtype=np.float32)
        (_, xd), (yb, yd) = _padded(x, offset), _padded(y0, 3 - offset)
        cs.conv_spmv(plan, xd, yd, batch=batch)
        torch.cuda.synchronize()
        _check(yd.cpu().numpy(), *oracle.conv(m, n, k, s, p, x, K, batch=batch, want_scale=True), (shape, batch))
        edge = yb.cpu().numpy()
        assert np.all(edge[:3 - offset] == 7.0) and np.all(edge[3 - offset + y0.size:] == 7.0)
    plan.close()


@pytest.mark.parametrize("shape,channels,batch", [
    ((40, 33, 3, 1, 1), 37, 1), ((40, 33, 5, 2, 2), 2, 3), ((40, 33, 3, 1, 1), 16, 6), ((20, 23, 13, 1, 12), 5, 7),
    ((40, 33, 1, 1, 0), 3, 2), ((9, 300, 4, 3, 1), 50, 5), ((21, 17, 2, 1, 1), 4, 19),
])
def test_channel_sums_in_row_groups_follow_the_descriptors(shape, channels, batch):
    """Batches the tiled channel sum does not take: the waves of a workgroup deal the channels out
    among themselves.  Two descriptors are edited (a smaller rectangle, an emptied row)."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(channels)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    x = rng.standard_normal(channels * m * n * batch).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()), channels=channels)
    assert plan.variant(batch).startswith("compact_gather")
    desc = oracle.compact_rows(m, n, k, s, p).copy()
    mid = plan.rows // 2
    w = int(np.uint32(desc[mid, 1]))
    r1 = w >> 8 & 255
    desc[mid, 1] = np.uint32(w - (1 << 8) if r1 > 1 else w).view(np.int32)
    desc[mid + 1] = 0
    plan.row_desc.copy_(torch.from_numpy(desc).to(device()))
    y = torch.full((plan.rows * batch,), float("nan"), dtype=torch.float32, device=device())
    cs.conv_spmv(plan, torch.from_numpy(x).to(device()), y, batch=batch)
    torch.cuda.synchronize()
    ref, scale = np.zeros((plan.rows, batch)), np.zeros((plan.rows, batch))
    for c in range(channels):
        rp, ci, va = oracle.compact_decode(n, k, desc, K[c * k * k:(c + 1) * k * k])
        T = scipy.sparse.csr_matrix((va.astype(np.float64), ci, rp), shape=(plan.rows, m * n))
        xc = x[c * m * n * batch:(c + 1) * m * n * batch].reshape(m * n, batch).astype(np.float64)
        ref += T @ xc
        scale += abs(T) @ np.abs(xc)
    _check(y.cpu().numpy(), ref.reshape(-1), scale.reshape(-1), (shape, channels, batch))
    plan.close()


def _launch_per_channel_error(K, channels, lanes, samples=4000):
    """2-norm error of float32 sums over `channels` channels with the kernels K, each channel summed by
    `lanes` chains of fused multiply-adds and a tree, then added to the sum of the channels before.  (The
    error depends on the kernels by some 7 %, on the pixels by the root of their number: 2 %.)"""
    rng = np.random.default_rng(2)
    total, ref = np.zeros(samples, np.float32), np.zeros(samples)
    for w in K.reshape(channels, -1):
        x = rng.standard_normal((w.size, samples)).astype(np.float32)
        parts = [np.zeros(samples, np.float32) for _ in range(lanes)]
        for t in range(w.size):
            parts[t % lanes] = (np.float64(w[t]) * x[t] + parts[t % lanes]).astype(np.float32)
        while len(parts) > 1:
            parts = [a + b for a, b in zip(parts[::2], parts[1::2])]
        total = total + parts[0]
        ref = ref + w.astype(np.float64) @ x
    return np.linalg.norm(total - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("shape,channels,batch,lanes", [     # lanes: k * k taps, at most 8 in a chain
    ((300, 300, 3, 1, 1), 64, 1, 2), ((300, 300, 2, 1, 0), 100, 2, 1), ((200, 180, 9, 1, 4), 16, 5, 16), ((200, 180, 7, 1, 3), 24, 3, 8),
    ((100, 90, 5, 1, 2), 20, 10, 4), ((200, 180, 11, 1, 5), 16, 1, 16), ((30, 40, 3, 1, 1), 120, 6, 2),
])
def test_channel_sums_in_row_groups_are_as_exact_as_a_launch_per_channel(shape, channels, batch, lanes):
    """All channels in one launch of the row groups: within 5 % (the scatter of the samples) of the
    error of a launch per channel; one chain per lane through all channels is up to twice as far off."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(channels)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    x = rng.standard_normal(channels * m * n * batch).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()), channels=channels)
    assert plan.variant(batch).startswith("compact_gather_"), plan.variant(batch)
    y = cs.conv_spmv(plan, torch.from_numpy(x).to(device()), batch=batch)
    torch.cuda.synchronize()
    ref, scale = oracle.conv_channels(m, n, k, s, p, x, K, channels, batch=batch, want_scale=True)
    got = y.cpu().numpy()
    _check(got, ref, scale, (shape, batch))
    ref = ref.astype(np.float64)
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1.05 * _launch_per_channel_error(K, channels, lanes)
    plan.close()


@pytest.mark.parametrize("k,s", [(4, 1), (13, 1), (12, 1), (10, 1), (1, 2), (4, 2), (9, 2), (13, 2), (1, 3), (3, 3), (7, 3), (13, 3),
                                 (2, 4), (4, 4), (5, 4), (11, 4), (17, 4)])
def test_pushed_lines_at_the_edges(k, s):
    """Input lines pushed into the output lines they reach: every number of output lines in flight,
    padding from none to k - 1, planes that end inside a window, a wave's part, a strip; an infinite
    kernel number stays out of the rows that do not hold its tap."""
    rng = np.random.default_rng(100 * k + s)
    for i, (m, n, p, batch) in enumerate(((k + 3, 70, 0, 4), (61, 33, k // 2, 16), (40 + s, 130, k - 1, 1), (k, 66 + k, 0, 9), (90, 41, k // 3, 5))):
        shape = (max(m, k), max(n, k), k, s, p)
        m, n = shape[:2]
        K = rng.standard_normal(k * k).astype(np.float32)
        if i == 2 and k > 1:
            K[0] = np.inf                              # the top left tap: border rows do not hold it
        x = rng.standard_normal(m * n * batch).astype(np.float32)
        plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()))
        cs.conv_plan_set_march_min_jobs(plan, 1)
        assert "_push%d_" % -(-k // s) in plan.variant(batch)
        y = torch.full((plan.rows * batch,), float("nan"), dtype=torch.float32, device=device())
        cs.conv_spmv(plan, torch.from_numpy(x).to(device()), y, batch=batch)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        if np.isinf(K[0]):
            rp, ci, va = oracle.csr(*shape, K)
            holds = np.add.reduceat(np.append(np.isinf(va), 0), rp[:-1]) * (np.diff(rp) > 0) > 0
            rows = got.reshape(-1, batch)
            assert holds.any() and not holds.all() and not np.isfinite(rows[holds]).any() and np.isfinite(rows[~holds]).all()
        else:
            _check(got, *oracle.conv(m, n, k, s, p, x, K, batch=batch, want_scale=True), (shape, batch))
        plan.close()


@pytest.mark.parametrize("kind,shape,batch,channels,want", [
    ("compact", (553, 440, 11, 2, 5), 28, 1, "compact_described_"), ("compact", (525, 510, 7, 3, 6), 36, 1, "compact_described_"),
    ("compact", (359, 277, 9, 1, 4), 12, 1, "compact_rect_"), ("compact", (420, 582, 11, 1, 5), 16, 1, "_ring"),
    ("compact", (205, 192, 1, 4, 0), 71, 10, "compact_gather_"), ("compact", (450, 559, 5, 4, 2), 36, 1, "compact_gather_"),
    ("csr", (393, 379, 11, 1, 0), 40, 1, "lds_march_28x32"), ("csr", (477, 694, 8, 1, 0), 3, 1, "lds_march_"),
    ("csr", (413, 252, 2, 1, 0), 32, 1, "lds_tile_7x64"), ("csr", (247, 335, 4, 1, 2), 3, 4, "gather_"),
    ("csc", (340, 367, 3, 2, 1), 160, 1, "block_"), ("csc", (340, 367, 3, 2, 1), 40, 1, "block_"),
    ("csc", (340, 367, 3, 2, 1), 32, 1, "lds_tile_"), ("csc", (340, 367, 3, 2, 1), 18, 1, "gather_"),
    ("csr", (475, 679, 5, 1, 2), 40, 1, "lds_march_staged_"), ("csr", (128, 128, 5, 1, 2), 128, 1, "block_"),
    ("csc", (93, 124, 5, 1, 0), 160, 1, "lds_tile_"), ("csc", (37, 48, 12, 3, 6), 178, 1, "gather_"),
])
def test_products_on_both_sides_of_the_dispatch_rules(kind, shape, batch, channels, want):
    """Lanes, kernels and tiles that the default dispatch gives shapes of ordinary size."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(29)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    Kd = torch.from_numpy(K).to(device())
    plan = (cs.conv_compact_build(*shape, Kd, channels=channels) if kind == "compact" else cs.conv_csc_build(*shape, Kd)
            if kind == "csc" else cs.conv_csr_build_channels(*shape, Kd, channels))
    assert want in plan.variant(batch), plan.variant(batch)
    x = rng.standard_normal(plan.cols * batch).astype(np.float32)
    y = torch.full((plan.rows * batch,), float("nan"), dtype=torch.float32, device=device())
    cs.conv_spmv(plan, torch.from_numpy(x).to(device()), y, batch=batch)
    torch.cuda.synchronize()
    ref = (oracle.conv_t(m, n, k, s, p, x, K, batch=batch, want_scale=True) if kind == "csc" else
           oracle.conv_channels(m, n, k, s, p, x, K, channels, batch=batch, want_scale=True))
    _check(y.cpu().numpy(), *ref, (kind, shape, batch))
    plan.close()


@pytest.mark.parametrize("shape,batch,want", [
    ((512, 512, 7, 2, 3), 12, "compact_rect_"), ((713, 1068, 11, 4, 5), 64, "_push3_float4"), ((333, 504, 13, 1, 0), 3, "_push13_scalar"),
    ((553, 440, 11, 2, 5), 28, "_ring"), ((1176, 1484, 13, 2, 6), 1, "_ring"), ((243, 337, 7, 1, 3), 15, "compact_rect_"),
    ((262, 253, 9, 1, 4), 11, "compact_rect_"), ((418, 445, 5, 1, 2), 6, "compact_rect_"),
])
def test_products_of_few_workgroups_sum_line_by_line(shape, batch, want):
    """Marching and pushing launches that take the place of row groups: the taps of a line are summed
    before the lines are, within 5 % (the scatter of the samples) of the error that has; one chain
    through all taps is 1.8 to 2.4 times as far off."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(31)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = cs.conv_compact_build(*shape, torch.from_numpy(K).to(device()))
    assert want in plan.variant(batch), plan.variant(batch)
    x = rng.standard_normal(plan.cols * batch).astype(np.float32)
    y = torch.full((plan.rows * batch,), float("nan"), dtype=torch.float32, device=device())
    cs.conv_spmv(plan, torch.from_numpy(x).to(device()), y, batch=batch)
    torch.cuda.synchronize()
    ref, scale = oracle.conv(m, n, k, s, p, x, K, batch=batch, want_scale=True)
    got = y.cpu().numpy()
    _check(got, ref, scale, (shape, batch))
    # 20 000 of the outputs against sums in 64 bits
    i, j, c = (rng.integers(0, top, 20000) for top in (plan.m_out, plan.n_out, batch))
    xp = np.zeros((m + 2 * p, n + 2 * p, batch), np.float32)
    xp[p:p + m, p:p + n] = x.reshape(m, n, batch)
    exact = sum(np.float64(K[a * k + b]) * xp[i * s + a, j * s + b, c] for a in range(k) for b in range(k))
    error = np.linalg.norm(got.reshape(plan.m_out, plan.n_out, batch)[i, j, c] - exact) / np.linalg.norm(exact)
    assert error <= 1.05 * _launch_per_channel_error(K, k, 1), error
    plan.close()


def test_rows_at_the_last_entry_numbers():
    """2^31 - 2 entries: the row groups step past the end of the last rows, up to 80 entries at once, where an
    entry number would leave the range of int.  The last output lines against sums in 64 bits."""
    m, n, k, s, p = shape = (3425, 7756, 9, 1, 2)
    assert cs.conv_nnz(*shape) == 2 ** 31 - 2
    mo, no = cs.conv_out_shape(*shape)
    g = torch.Generator(device="cuda").manual_seed(5)
    K = torch.randn(k * k, device=device(), generator=g)

    def last_lines(x, batch, lines=6):         # of y = T x
        pad = torch.zeros(m + 2 * p - (mo - lines), n + 2 * p, batch, dtype=torch.float64, device=device())
        pad[:-p, p:-p] = x.view(m, n, batch)[mo - lines - p:].double()
        y, scale = (torch.zeros(lines, no, batch, dtype=torch.float64, device=device()) for _ in range(2))
        for a in range(k):
            for b in range(k):
                y += K[a * k + b].double() * pad[a:a + lines, b:b + no]
                scale += K[a * k + b].double().abs() * pad[a:a + lines, b:b + no].abs()
        return y.reshape(-1), scale.reshape(-1)

    def check(y, x, batch, what):
        ref, scale = last_lines(x, batch)
        assert not bool(torch.isnan(y).any()), what
        assert bool(((y[-ref.numel():].double() - ref).abs() <= REL_TOL * scale).all()), what

    plan = cs.conv_csr_build(*shape, K)
    for batch in (1, 4):
        x = torch.randn(m * n * batch, device=device(), generator=g)
        y = torch.full((plan.rows * batch,), float("nan"), device=device())
        multi = cs.ConvMulti([plan], [x], [y], batch=batch)
        multi.apply()
        check(y, x, batch, ("multi", batch))
        multi.close()
    plan.close()
    del plan, multi
    torch.cuda.empty_cache()
    plan = cs.conv_csc_build(*shape, K)
    x = torch.randn(m * n, device=device(), generator=g)
    y = torch.full((plan.cols,), float("nan"), device=device())
    cs.conv_spmv_from_csc(plan, x, y)
    check(y, x, 1, "from csc")
    keep_to_the_scatter(plan, shape, 1, kernel=8)
    y.fill_(float("nan"))
    cs.conv_spmv_from_csc(plan, x, y)
    check(y, x, 1, "scatter")
    plan.close()
    del plan
    torch.cuda.empty_cache()
