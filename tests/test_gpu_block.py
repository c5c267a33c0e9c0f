"""Products in blocks of outputs with the batch on the lanes (apply_block_kernel.h), T and T^T, against the oracle."""
import numpy as np
import pytest
import scipy.sparse
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, device

pytestmark = pytest.mark.gpu

SHAPES = [("csr", k, s) for s in (1, 2) for k in (2, 3, 4, 5)] + [("csr", k, s) for s in (3, 4) for k in (3, 4, 5)] + \
    [("csc", k, 1) for k in (2, 3, 4, 5)] + [("csc", k, 2) for k in range(3, 11)] + \
    [("csc", k, 3) for k in range(4, 13)] + [("csc", k, 4) for k in range(5, 14)]


def _check(got, ref, scale, what):
    assert not np.any(np.isnan(got)), what
    assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= REL_TOL * scale), what


@pytest.mark.parametrize("storage,k,s", SHAPES)
def test_blocks_at_edges_and_paddings(storage, k, s):
    """Planes that end anywhere in a block, padding from none to more than the kernel, lanes full and partly idle,
    batches that are no multiple of 4, operands at any float address.  The first plane is the smallest one that the dispatch gives
    to blocks; the others are lines of pixels, which it may give to another kernel."""
    rng = np.random.default_rng(100 * k + s)
    conv = oracle.conv if storage == "csr" else oracle.conv_t
    for i, (p, batch) in enumerate(((0, 64), (k // 2, 125), (k - 1, 131), (k + 1, 49), (k // 2, 256))):
        planes = [(f * s + i, f * s - s + 2 * i + 1) for f in (16, 24, 32, 48, 64, 92, 120, 150, 180, 220)]
        m0, n0 = next((m, n) for m, n in planes
                      if cs.conv_dispatch_info(m, n, k, s, p, batch, int(storage == "csc")).kernel == 12)
        for m, n in ((m0, n0), (k + 2, 900 * s + i), (900 * s + i, k + 1), (k, 9 * s + i)):
            K = rng.standard_normal(k * k).astype(np.float32)
            plan = (cs.conv_csr_build if storage == "csr" else cs.conv_csc_build)(m, n, k, s, p, torch.from_numpy(K).to(device()))
            assert (m, n) != (m0, n0) or plan.variant(batch).startswith("block_")
            x = rng.standard_normal(plan.cols * batch).astype(np.float32)
            xb = torch.full((x.size + 4,), 7.0, device=device())
            yb = torch.full((plan.rows * batch + 8,), 7.0, device=device())
            xd, yd = xb[i % 4:i % 4 + x.size], yb[4 - i % 4:4 - i % 4 + plan.rows * batch]
            xd.copy_(torch.from_numpy(x))
            yd.fill_(float("nan"))
            cs.conv_spmv(plan, xd, yd, batch=batch)
            torch.cuda.synchronize()
            _check(yd.cpu().numpy(), *conv(m, n, k, s, p, x, K, batch=batch, want_scale=True), (m, n, p, batch))
            edge = yb.cpu().numpy()
            assert np.all(edge[:4 - i % 4] == 7.0) and np.all(edge[4 - i % 4 + plan.rows * batch:] == 7.0)
            plan.close()


@pytest.mark.parametrize("storage,shape,batch", [("csr", (60, 71, 3, 1, 1), 64), ("csr", (200, 183, 5, 2, 2), 112),
                                                 ("csc", (60, 71, 3, 1, 1), 126), ("csc", (90, 83, 5, 2, 2), 60),
                                                 ("csc", (190, 163, 7, 3, 3), 64), ("csc", (200, 190, 9, 2, 4), 64),
                                                 ("csr", (160, 163, 5, 3, 2), 64)])
def test_blocks_read_the_stored_arrays(storage, shape, batch):
    """Columns redirected after the build, entries moved between neighbouring rows, infinite values: the product follows the
    arrays; in image-border blocks too."""
    m, n, k, s, p = shape
    rng = np.random.default_rng(5)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan = (cs.conv_csr_build if storage == "csr" else cs.conv_csc_build)(*shape, torch.from_numpy(K).to(device()))
    assert plan.variant(batch).startswith("block_")
    x = rng.standard_normal(plan.cols * batch).astype(np.float32)
    xd = torch.from_numpy(x).to(device())
    before = cs.conv_spmv(plan, xd, batch=batch).cpu().numpy().reshape(-1, batch)
    ptr, idx, vals = (t.cpu().numpy().copy() for t in (plan.row_ptr, plan.col_idx, plan.vals))
    rows = rng.choice(plan.rows - 2, size=40, replace=False)
    rows = np.concatenate([rows[(np.diff(ptr)[rows] > 2) & (np.diff(ptr)[rows + 1] > 0)], [0]])
    for i, row in enumerate(rows):
        if i % 3 == 2:
            ptr[row + 1] -= 1                    # the row's last entry goes to the next row
        else:
            idx[ptr[row] + i % 2] = rng.integers(plan.cols)
    plan.row_ptr.copy_(torch.from_numpy(ptr))
    plan.col_idx.copy_(torch.from_numpy(idx))
    got = cs.conv_spmv(plan, xd, batch=batch).cpu().numpy().reshape(-1, batch)
    # (copies: abs() merges duplicates in place)
    T = scipy.sparse.csr_matrix((vals.astype(np.float64), idx.copy(), ptr.copy()), shape=(plan.rows, plan.cols))
    x2 = x.reshape(-1, batch).astype(np.float64)
    scale = abs(T) @ abs(x2)
    assert np.all(np.abs(got - T @ x2) <= REL_TOL * scale + 1e-30)
    changed = np.union1d(rows, rows + 1)
    same = np.setdiff1d(np.arange(plan.rows), changed)
    # (a wave with an edited row sums entry by entry: other roundings, no other result)
    assert np.all(np.abs(got[same] - before[same]) <= 2 * REL_TOL * scale[same])
    vals[ptr[rows[0]]] = np.inf
    plan.vals.copy_(torch.from_numpy(vals))
    hit = ~np.isfinite(cs.conv_spmv(plan, xd, batch=batch).cpu().numpy().reshape(-1, batch)).all(axis=1)
    assert list(np.flatnonzero(hit)) == [rows[0]]
    plan.close()


@pytest.mark.parametrize("storage", ["csr", "csc"])
def test_blocks_of_operands_just_below_four_gib(storage):
    """Byte offsets of 32 bits, unsigned: 3900 x 4000 pixels of 68 columns are 4.24e9 bytes, the first and the last 24 lines
    against float64 sums."""
    shape, batch, lines = (3900, 4000, 3, 1, 1), 68, 24
    m, n, k, s, p = shape
    g = torch.Generator(device=device()).manual_seed(6)
    K = torch.randn(k * k, device=device(), generator=g)
    plan = (cs.conv_csr_build if storage == "csr" else cs.conv_csc_build)(*shape, K)
    assert plan.variant(batch).startswith("block_") and 4 * plan.cols * batch > 0.98 * 2 ** 32
    x = torch.randn(plan.cols * batch, device=device(), generator=g)
    y = torch.full((plan.rows * batch,), float("nan"), device=device())
    cs.conv_spmv(plan, x, y, batch=batch)
    taps = K if storage == "csr" else K.flip(0)              # T^T at "same" padding: the kernel turned round
    for top in (True, False):
        pad = torch.zeros(lines + 2, n + 2, batch, dtype=torch.float64, device=device())
        if top:
            pad[1:, 1:-1] = x.view(m, n, batch)[:lines + 1]
        else:
            pad[:-1, 1:-1] = x.view(m, n, batch)[m - lines - 1:]
        got = y.view(m, n, batch)[:lines] if top else y.view(m, n, batch)[m - lines:]
        ref, scale = torch.zeros_like(got, dtype=torch.float64), torch.zeros_like(got, dtype=torch.float64)
        for a in range(k):
            for b in range(k):
                ref += taps[a * k + b].double() * pad[a:a + lines, b:b + n]
                scale += taps[a * k + b].double().abs() * pad[a:a + lines, b:b + n].abs()
        assert bool(((got.double() - ref).abs() <= REL_TOL * scale).all()), top
    assert not bool(torch.isnan(y).any())
    plan.close()
