"""Every kernel that items are compiled as: columns per lane, lanes per item, entries asked for at a time, with and without channels that
waves share.  Each is named as the dispatch names it and as the launch picks the entries by the rows; as built, and with columns
moved and entries handed to the next row.  Reference: scipy's product of the arrays as they are, in 64 bits."""
import numpy as np
import pytest
import scipy.sparse
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

# storage, shape, batch, columns, lanes, longest row (1, 4, 9 at once; 25 in fives; others in fours)
ONE = [
    ("csr", (6, 6, 1, 4, 2), 2, 1, 1, 1), ("csr", (7, 6, 2, 4, 1), 2, 1, 1, 4), ("csc", (208, 315, 9, 4, 0), 2, 1, 1, 9), ("csr", (6, 6, 3, 4, 0), 2, 1, 2, 9),
    ("csc", (212, 209, 13, 3, 0), 3, 1, 1, 25), ("csc", (136, 243, 13, 3, 0), 2, 1, 2, 25), ("csc", (255, 263, 13, 4, 0), 2, 1, 1, 16), ("csr", (7, 7, 4, 4, 0), 2, 1, 2, 16),
    ("csr", (7, 6, 5, 3, 0), 2, 1, 4, 25), ("csr", (7, 9, 6, 4, 0), 2, 1, 8, 36), ("csr", (175, 204, 13, 2, 0), 2, 1, 16, 169),
    ("csc", (142, 155, 2, 2, 0), 9, 4, 1, 1), ("csr", (160, 139, 2, 2, 0), 9, 4, 1, 4), ("csc", (29, 21, 7, 3, 0), 258, 4, 1, 9), ("csc", (51, 58, 6, 2, 0), 9, 4, 2, 9),
    ("csc", (29, 17, 13, 3, 0), 269, 4, 1, 25), ("csc", (27, 18, 13, 3, 0), 266, 4, 2, 25), ("csc", (17, 28, 7, 2, 0), 286, 4, 1, 16), ("csr", (20, 26, 4, 2, 5), 298, 4, 2, 16),
    ("csr", (47, 49, 4, 2, 2), 34, 4, 4, 16), ("csr", (60, 46, 5, 3, 4), 65, 4, 8, 25), ("csr", (145, 210, 6, 2, 3), 97, 4, 1, 36), ("csr", (60, 64, 8, 1, 4), 118, 4, 1, 64),
]
# shape, batch, channels, columns, lanes, ways
MANY = [
    ((29, 41, 1, 1, 2), 3, 2, 1, 1, 1), ((27, 40, 1, 1, 2), 3, 9, 1, 1, 2), ((11, 16, 1, 1, 2), 62, 2, 4, 1, 1), ((6, 6, 1, 1, 2), 170, 9, 4, 1, 2),
    ((321, 549, 3, 1, 4), 3, 2, 1, 1, 1), ((354, 379, 3, 1, 1), 2, 2, 1, 2, 1), ((9, 6, 3, 2, 4), 3, 2, 1, 4, 1), ((7, 6, 3, 2, 4), 3, 9, 1, 4, 2),
    ((344, 214, 3, 2, 4), 109, 2, 4, 1, 1), ((291, 326, 3, 2, 4), 41, 2, 4, 2, 1), ((7, 6, 3, 3, 4), 21, 3, 4, 4, 1), ((6, 6, 3, 2, 4), 13, 8, 4, 4, 2),
    ((32, 36, 2, 1, 3), 3, 2, 1, 1, 1), ((32, 55, 2, 1, 3), 2, 8, 1, 1, 2), ((241, 368, 4, 1, 2), 3, 2, 1, 2, 1), ((7, 9, 4, 4, 0), 1, 8, 1, 4, 2),
    ((8, 7, 5, 4, 0), 1, 2, 1, 8, 1), ((6, 6, 5, 2, 0), 1, 10, 1, 8, 2), ((7, 7, 6, 2, 0), 1, 2, 1, 16, 1), ((7, 7, 6, 2, 0), 1, 130, 1, 16, 16),
    ((6, 8, 2, 1, 3), 122, 3, 4, 1, 1), ((58, 33, 2, 1, 3), 5, 8, 4, 1, 2), ((84, 124, 4, 3, 0), 955, 2, 4, 2, 1), ((6, 6, 4, 3, 0), 10, 9, 4, 4, 2),
    ((6, 7, 5, 2, 0), 7, 2, 4, 8, 1), ((6, 6, 5, 2, 0), 5, 35, 4, 8, 8), ((6, 6, 6, 2, 0), 9, 2, 4, 16, 1), ((9, 6, 6, 4, 0), 5, 70, 4, 16, 16),
]


def _edited(rng, ptr, idx, cols):
    """Another matrix in the same arrays: columns moved, rows emptied, an entry handed to the row after (never more than a row of two)."""
    ptr, idx = ptr.copy(), idx.copy()
    idx[rng.choice(idx.size, size=min(40, idx.size))] = rng.integers(0, cols, size=min(40, idx.size))
    rows = np.arange(1, ptr.size - 1, max(2, (ptr.size - 2) // 20))
    for row in rows:
        ptr[row] = ptr[row - 1] if row % 3 == 0 else max(ptr[row] - 1, ptr[row - 1])
    return ptr, idx


def _run(plan, arrays, vals, batch, rng, what):
    """The plan's product, operands at every alignment, against the matrices that its arrays hold."""
    x = rng.standard_normal((plan.cols, batch)).astype(np.float32)
    buf = torch.full((plan.rows * batch + 8,), 7.0, dtype=torch.float32, device=device())
    for i, (ptr, idx) in enumerate(arrays):
        offset = 3 - i
        xd = torch.empty(x.size + 4, dtype=torch.float32, device=device())[offset:offset + x.size]
        xd.copy_(torch.from_numpy(x.reshape(-1)))
        y = buf[i + 1:i + 1 + plan.rows * batch].fill_(float("nan"))
        plan.row_ptr.copy_(torch.from_numpy(ptr.astype(np.int32)))
        plan.col_idx.copy_(torch.from_numpy(idx.astype(np.int32)))
        cs.conv_spmv(plan, xd, y, batch=batch)
        got = y.cpu().numpy().astype(np.float64).reshape(plan.rows, batch)
        plane = plan.cols // plan.channels
        want, bound = np.zeros(got.shape), np.zeros(got.shape)
        for c in range(plan.channels):
            A = scipy.sparse.csr_matrix((vals[c], idx, ptr), shape=(plan.rows, plane)).astype(np.float64)
            xc = x[c * plane:(c + 1) * plane].astype(np.float64)
            want += A @ xc
            bound += abs(A) @ abs(xc)
        assert np.all(np.abs(got - want) <= REL_TOL * bound), (what, i)
        edge = buf.cpu().numpy()
        assert np.all(edge[:i + 1] == 7.0) and np.all(edge[i + 1 + got.size:] == 7.0), (what, i)
        buf.fill_(7.0)


@pytest.mark.gpu
@pytest.mark.parametrize("storage,shape,batch,columns,lanes,longest", ONE)
def test_one_channel(storage, shape, batch, columns, lanes, longest):
    m, n, k, s, p = shape
    assert longest == (k if storage == "csr" else -(-k // s)) ** 2
    rng = np.random.default_rng(74)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = (cs.conv_csr_build if storage == "csr" else cs.conv_csc_build)(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch) == "gather_g%d_%s_items" % (lanes, "float4" if columns == 4 else "scalar")
    ptr, idx, vals = oracle.csr(*shape, K)
    if storage == "csc":
        T = scipy.sparse.csr_matrix((vals, idx, ptr), shape=(plan.m_out * plan.n_out, m * n)).T.tocsr()
        T.sort_indices()
        ptr, idx, vals = T.indptr, T.indices, T.data
    _run(plan, [(ptr, idx), _edited(rng, ptr, idx, plan.cols)], [vals], batch, rng, (storage, shape, batch))
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("shape,batch,channels,columns,lanes,ways", MANY)
def test_channels(shape, batch, channels, columns, lanes, ways):
    m, n, k, s, p = shape
    rng = np.random.default_rng(75)
    K = rng.standard_normal((channels, k * k)).astype(np.float32)
    plan = cs.conv_csr_build_channels(*shape, torch.from_numpy(K.reshape(-1)).to(device()), channels)
    name = "gather_g%d_%s_items%s" % (lanes, "float4" if columns == 4 else "scalar", "_%d_ways" % ways if ways > 1 else "")
    assert plan.variant(batch) == "%s_%d_channels" % (name, channels)
    ptr, idx, _ = oracle.csr(*shape, K[0])
    vals = [oracle.csr(*shape, K[c])[2] for c in range(channels)]
    _run(plan, [(ptr, idx), _edited(rng, ptr, idx, plan.cols // channels)], vals, batch, rng, (shape, batch, channels))
    plan.close()


@pytest.mark.parametrize("storage,shape,batch,columns,lanes,longest", ONE)
def test_dispatch(storage, shape, batch, columns, lanes, longest):
    d = cs.conv_dispatch_info(*shape, batch, int(storage == "csc"))
    assert (d.kernel, d.strip, d.columns_per_lane, d.lanes_per_row) == (int(columns == 4), -(-batch // columns), columns, lanes)


@pytest.mark.parametrize("shape,batch,channels,columns,lanes,ways", MANY)
def test_dispatch_of_channels(shape, batch, channels, columns, lanes, ways):
    d = cs.conv_dispatch_info(*shape, batch, 0, channels)
    assert (d.kernel, d.strip, d.columns_per_lane, d.lanes_per_row, d.threads) == (int(columns == 4), -(-batch // columns), columns, lanes, 64 * ways)
    assert d.lds_bytes == (ways * (64 // lanes) * columns * 8 if ways > 1 else 0)
