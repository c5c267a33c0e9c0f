"""Row groups with the chunks of a row side by side on the lanes: rows of 1 to 169 entries, full and ragged batches, operands
at any alignment, edited arrays, channels dealt to waves.  (Every compiled kernel by name: test_gpu_item_kernels.py.)
Reference: the sliding-window oracle, and scipy's product of the arrays as they are."""
import numpy as np
import pytest
import scipy.sparse
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

pytestmark = pytest.mark.gpu


def _operands(size_x, size_y, offset):
    buf = torch.full((size_y + 8,), 7.0, dtype=torch.float32, device=device())
    x = torch.empty(size_x + 8, dtype=torch.float32, device=device())[offset:offset + size_x]
    return x, buf, buf[3 - offset:3 - offset + size_y].fill_(float("nan"))


def _check(y, buf, offset, ref, scale, what):
    got, edge = y.cpu().numpy().astype(np.float64), buf.cpu().numpy()
    assert np.all(np.abs(got - ref) <= REL_TOL * scale), what           # (a NaN left over is not)
    assert np.all(edge[:3 - offset] == 7.0) and np.all(edge[3 - offset + got.size:] == 7.0), what


# rows of 1, 4, 9, 25 and up to 169 entries, borders of p >= k; at one batch of each at least items take the product
@pytest.mark.parametrize("storage,shape,batches", [
    ("csr", (64, 61, 1, 1, 0), (33, 131)), ("csr", (150, 140, 2, 2, 1), (20, 31)), ("csr", (161, 158, 3, 1, 1), (2, 3, 20)),
    ("csr", (90, 81, 5, 2, 2), (20, 31)), ("csr", (90, 91, 6, 3, 5), (40, 131)), ("csr", (70, 75, 7, 3, 3), (70, 101)),
    ("csr", (60, 70, 8, 1, 4), (44, 74)), ("csr", (66, 65, 11, 2, 5), (66, 200)), ("csr", (90, 101, 13, 1, 6), (100,)),
    ("csr", (140, 139, 6, 3, 8), (60, 101)), ("csc", (150, 161, 1, 2, 0), (60, 101)), ("csc", (81, 70, 3, 3, 1), (51, 90)),
    ("csc", (60, 61, 6, 1, 3), (85,)), ("csc", (120, 110, 11, 4, 5), (24,)), ("csc", (64, 85, 13, 2, 6), (61,)),
])
def test_items(storage, shape, batches):
    m, n, k, s, p = shape
    rng = np.random.default_rng(71)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = (cs.conv_csr_build if storage == "csr" else cs.conv_csc_build)(*shape, torch.from_numpy(K).to(device()))
    rp, ci, va = oracle.csr(*shape, K)
    T = scipy.sparse.csr_matrix((va, ci, rp), shape=(plan.m_out * plan.n_out, m * n))
    if storage == "csc":
        T = T.T.tocsr()
        T.sort_indices()
    # another matrix in the same arrays: columns moved, an entry handed to the next row, a row emptied
    idx, ptr = T.indices.copy(), T.indptr.copy()
    idx[rng.choice(idx.size, size=40)] = rng.integers(0, plan.cols, size=40)
    for row in rng.choice(plan.rows - 2, size=20, replace=False) + 1:
        ptr[row] = ptr[row - 1] if row % 2 else max(ptr[row] - 1, ptr[row - 1])
    edited = scipy.sparse.csr_matrix((T.data, idx, ptr), shape=T.shape)
    ran = set()
    for i, batch in enumerate(batches):
        offset = i % 4
        ran.add(plan.variant(batch).endswith("_items"))
        x = rng.standard_normal((plan.cols, batch))
        xd, buf, yd = _operands(plan.cols * batch, plan.rows * batch, offset)
        xd.copy_(torch.from_numpy(x.reshape(-1)))
        x = xd.cpu().numpy().astype(np.float64).reshape(plan.cols, batch)
        for matrix, columns, rows in ((T, T.indices, T.indptr), (edited, idx, ptr)):
            plan.col_idx.copy_(torch.from_numpy(columns))
            plan.row_ptr.copy_(torch.from_numpy(rows))
            cs.conv_spmv(plan, xd, yd.fill_(float("nan")), batch=batch)
            torch.cuda.synchronize()
            A = matrix.astype(np.float64)
            _check(yd, buf, offset, (A @ x).reshape(-1), (abs(A) @ abs(x)).reshape(-1), (shape, batch, matrix is T))
    assert True in ran
    plan.close()


def test_items_keep_infinite_values_to_their_rows():
    shape, batch = (80, 84, 7, 3, 3), 60
    m, n, k, s, p = shape
    rng = np.random.default_rng(72)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = cs.conv_csr_build(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch).endswith("_items")
    x = rng.standard_normal((m * n, batch)).astype(np.float32)
    x[777, 5], x[1000, 59] = np.inf, np.nan
    y = cs.conv_spmv(plan, torch.from_numpy(x.reshape(-1)).to(device()), batch=batch).cpu().numpy().reshape(-1, batch)
    rp, ci, _ = oracle.csr(*shape, K)
    holds = np.zeros_like(y, dtype=bool)
    for pixel, column in ((777, 5), (1000, 59)):
        rows = np.searchsorted(rp, np.flatnonzero(ci == pixel), side="right") - 1
        holds[rows, column] = True
    assert np.array_equal(~np.isfinite(y), holds) and holds.any()
    plan.close()


@pytest.mark.parametrize("shape,batch,channels", [
    ((120, 121, 1, 1, 0), 22, 9), ((40, 41, 1, 1, 0), 16, 130), ((30, 31, 9, 3, 8), 2, 136), ((17, 18, 3, 1, 1), 1, 33), ((19, 20, 3, 2, 1), 60, 16),
    ((20, 28, 6, 3, 3), 60, 65), ((53, 31, 5, 2, 2), 7, 8), ((17, 22, 11, 1, 5), 14, 14), ((37, 57, 4, 4, 3), 1, 170), ((16, 16, 13, 1, 6), 3, 2),
])
def test_channels_dealt_to_waves(shape, batch, channels):
    m, n, k, s, p = shape
    rng = np.random.default_rng(73)
    K = rng.standard_normal(channels * k * k).astype(np.float32)
    plan = cs.conv_csr_build_channels(*shape, torch.from_numpy(K).to(device()), channels)
    assert "_items" in plan.variant(batch), plan.variant(batch)
    x = rng.standard_normal(plan.cols * batch).astype(np.float32)
    ref, scale = oracle.conv_channels(m, n, k, s, p, x, K, channels, batch=batch, want_scale=True)
    for offset in (0, 1):
        xd, buf, yd = _operands(x.size, plan.rows * batch, offset)
        xd.copy_(torch.from_numpy(x))
        cs.conv_spmv(plan, xd, yd, batch=batch)
        torch.cuda.synchronize()
        _check(yd, buf, offset, ref.astype(np.float64), scale, (shape, batch, channels))
    plan.close()
