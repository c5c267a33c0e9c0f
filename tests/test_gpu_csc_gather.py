"""GPU parity of the gathering product from the column-compressed arrays (conv_spmv_from_csc): against the
sliding-window oracle where the arrays are as built, against scipy's product where they were edited."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs

from gpu_util import build_plan_t, device, median_us
from test_csc_gather_rule import gather_info

pytestmark = pytest.mark.gpu

# fp32 sums of at most 169 products, a line's taps first: |error| <= 1e-5 of the sum of |products| (observed below 4e-7)
REL_TOL = 1e-5


def plan_of(shape, K, batch):
    plan = build_plan_t(shape, K)
    cs.conv_plan_set_march_min_jobs(plan, 1)
    assert gather_info(*shape, batch, jobs=1)["kernel"] == 11
    return plan


def inputs(shape, batch, seed):
    m, n, k, s, p = shape
    rng = np.random.default_rng(seed)
    return rng.standard_normal(m * n * batch).astype(np.float32), rng.standard_normal(k * k).astype(np.float32)


@pytest.mark.parametrize("shape,batch", [
    # every number of lines in flight, stride 1, each lane layout and both depths; strips of one output more or less
    ((150, 260, 1, 1, 0), 16), ((70, 65, 2, 1, 1), 4), ((90, 129, 3, 1, 1), 1), ((40, 63, 4, 1, 0), 7), ((64, 64, 5, 1, 2), 16),
    ((75, 80, 6, 1, 3), 33), ((100, 127, 7, 1, 3), 16), ((61, 66, 7, 1, 6), 2), ((93, 70, 8, 1, 4), 12), ((90, 97, 9, 1, 4), 5),
    ((100, 95, 10, 1, 0), 9), ((101, 90, 11, 1, 5), 17), ((120, 111, 12, 1, 11), 8), ((110, 113, 13, 1, 6), 4), ((130, 98, 13, 1, 6), 1),
    # planes lower than a window, one output column, one line of outputs
    ((3, 200, 7, 1, 3), 16), ((300, 9, 5, 1, 4), 16), ((7, 300, 7, 1, 0), 16), ((300, 7, 7, 1, 0), 16),
    # strides that divide k and that do not, remainders of the image below and right of the last window
    ((200, 301, 2, 2, 0), 16), ((151, 164, 3, 2, 1), 16), ((180, 190, 5, 2, 2), 4), ((97, 130, 5, 3, 1), 19), ((200, 203, 7, 2, 3), 1),
    ((150, 171, 7, 4, 3), 6), ((203, 202, 9, 3, 8), 8), ((201, 150, 11, 4, 5), 4), ((200, 190, 13, 2, 6), 3), ((170, 161, 13, 4, 12), 16),
    ((160, 259, 4, 4, 0), 64), ((203, 301, 3, 3, 0), 24),
])
def test_gather_matches_the_oracle_and_itself(shape, batch):
    x, K = inputs(shape, batch, 3)
    plan = plan_of(shape, K, batch)
    xd = torch.from_numpy(x).to(device())
    y = torch.full((plan.cols * batch + 8,), 7.0, dtype=torch.float32, device=device())
    offset = 1 if batch % 2 else 4                                  # results on a 4-byte and on a 16-byte boundary
    out = y[offset:offset + plan.cols * batch]
    cs.conv_spmv_from_csc(plan, xd, out, batch=batch)
    again = cs.conv_spmv_from_csc(plan, xd, batch=batch)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert np.all(got[:offset] == 7.0) and np.all(got[offset + plan.cols * batch:] == 7.0)
    got = got[offset:offset + plan.cols * batch]
    assert np.array_equal(got, again.cpu().numpy())                 # a fixed order of sums
    ref, scale = oracle.conv(*shape, x, K, batch=batch, want_scale=True)
    assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= REL_TOL * scale)
    plan.close()


def edited_product(shape, batch, edit, seed=5):
    """The product after edit(col_ptr, row_idx, vals) on host copies of the arrays; scipy's with the same."""
    import scipy.sparse as sp
    x, K = inputs(shape, batch, seed)
    plan = plan_of(shape, K, batch)
    cp, ri, va = (np.array(a) for a in oracle.csc(*shape, K))
    edit(cp, ri, va, plan)
    plan.row_ptr.copy_(torch.from_numpy(cp.astype(np.int32)))
    plan.col_idx.copy_(torch.from_numpy(ri.astype(np.int32)))
    plan.vals.copy_(torch.from_numpy(va.astype(np.float32)))
    y = torch.full((plan.cols * batch,), float("nan"), dtype=torch.float32, device=device())
    cs.conv_spmv_from_csc(plan, torch.from_numpy(x).to(device()), y, batch=batch)
    torch.cuda.synchronize()
    T = sp.csc_matrix((va.astype(np.float64), ri, cp), shape=(plan.cols, plan.rows))
    X = x.reshape(-1, batch).astype(np.float64)
    plan.close()
    return y.cpu().numpy().reshape(-1, batch), T @ X, abs(T) @ np.abs(X)


@pytest.mark.parametrize("shape,batch", [((96, 180, 7, 1, 3), 16), ((130, 150, 3, 1, 1), 18), ((120, 133, 5, 2, 2), 5), ((140, 150, 9, 4, 4), 1)])
def test_gather_of_edited_arrays(shape, batch):
    """Entries sent near and far, to outputs that other workgroups own and to the first outputs of
    workgroups; values changed; an entry moved to the next column (two column pointers in error)."""
    m, n, k, s, p = shape
    d = gather_info(*shape, batch, jobs=1)
    mo, no = oracle.out_shape(*shape)
    rng = np.random.default_rng(8)

    def edit(cp, ri, va, plan):
        def entry(col):
            return int(rng.integers(cp[col], cp[col + 1]))

        full = np.flatnonzero(np.diff(cp) > 1)
        for target in (0, plan.cols - 1, min(d["segment"], mo - 1) * no, min(d["strip"], no - 1), int(rng.integers(plan.cols))):
            col = int(rng.choice(full))
            if target not in ri[cp[col]:cp[col + 1]]:
                ri[entry(col)] = target
        va[entry(int(rng.choice(full)))] = 3.5
        col = int(full[len(full) // 2])                              # its last entry now belongs to the next column
        if cp[col + 2] - cp[col + 1] < (-(-k // s)) ** 2 and ri[cp[col + 1] - 1] not in ri[cp[col + 1]:cp[col + 2]]:
            cp[col + 1] -= 1
    got, want, scale = edited_product(shape, batch, edit)
    assert np.all(np.abs(got - want) <= REL_TOL * scale + 1e-30)


def test_gather_of_arrays_with_every_column_edited():
    """Every workgroup has to sum its outputs again, and each has entries for the others."""
    def edit(cp, ri, va, plan):
        rng = np.random.default_rng(9)
        for col in range(plan.rows):
            e = int(cp[col])
            target = int(rng.integers(plan.cols))
            if cp[col + 1] > e and target not in ri[e:cp[col + 1]]:
                ri[e] = target
    got, want, scale = edited_product((80, 90, 5, 1, 2), 9, edit)
    assert np.all(np.abs(got - want) <= REL_TOL * scale + 1e-30)


@pytest.mark.parametrize("shape,batch", [((60, 150, 7, 1, 3), 16), ((80, 90, 5, 2, 2), 2)])
def test_an_infinite_pixel_reaches_only_its_windows(shape, batch):
    m, n, k, s, p = shape
    x, K = inputs(shape, batch, 11)
    K[K == 0] = 1.0
    x = x.reshape(m, n, batch)
    for i, j in ((0, 0), (m - 1, n - 1), (m // 2, 63), (m // 2, 64)):
        x[i, j, 0] = np.inf
    x[m // 3, n // 2, batch - 1] = np.nan
    plan = plan_of(shape, K, batch)
    y = cs.conv_spmv_from_csc(plan, torch.from_numpy(x.reshape(-1)).to(device()), batch=batch)
    torch.cuda.synchronize()
    ref = oracle.conv(*shape, x.reshape(-1), K, batch=batch)
    got = y.cpu().numpy()
    assert np.array_equal(np.isfinite(got), np.isfinite(ref)) and np.array_equal(np.isnan(got), np.isnan(ref))
    plan.close()


@pytest.mark.parametrize("edit", ["one", "every column"])
def test_edited_arrays_cost_no_more_than_a_scatter(edit):
    """Columns that are not as built are left to the scatter, which takes three to four times as long as the gather at this shape
    whatever the arrays hold: six times bounds the two together (every workgroup's outputs summed again took 70)."""
    shape, batch = (1024, 1024, 7, 1, 3), 16
    x, K = inputs(shape, batch, 12)
    plan, other = build_plan_t(shape, K), build_plan_t(shape, K)
    xd = torch.from_numpy(x).to(device())
    y = torch.empty(plan.cols * batch, device=device())
    as_built = median_us(lambda: cs.conv_spmv_from_csc(plan, xd, y, batch=batch))
    cols = slice(500 * 1024 + 37, 500 * 1024 + 38) if edit == "one" else slice(0, plan.rows)
    first = plan.row_ptr[:-1][cols].long()
    swapped = plan.col_idx[first + 1].clone()                        # the first two entries of a column change places
    plan.col_idx[first + 1] = plan.col_idx[first]
    plan.col_idx[first] = swapped
    edited = median_us(lambda: cs.conv_spmv_from_csc(plan, xd, y, batch=batch))
    assert edited <= 6 * as_built, (as_built, edited)
    untouched = median_us(lambda: cs.conv_spmv_from_csc(other, xd, y, batch=batch))     # another plan is not slowed by it
    assert untouched <= 1.5 * as_built, (as_built, untouched)
    plan.close()
    other.close()


@pytest.mark.parametrize("shape,batch", [((96, 180, 7, 1, 3), 16), ((130, 150, 3, 1, 1), 18), ((120, 133, 5, 2, 2), 5),
                                         ((140, 150, 9, 4, 4), 1), ((150, 140, 1, 1, 0), 20), ((200, 190, 4, 2, 1), 3)])
def test_an_infinite_pixel_does_not_reach_what_its_edited_column_left(shape, batch):
    """Of pixels that are infinite, the entries are sent elsewhere: the outputs they have left stay finite."""
    import scipy.sparse as sp
    m, n, k, s, p = shape
    x, K = inputs(shape, batch, 15)
    K[K == 0] = 1.0
    plan = plan_of(shape, K, batch)
    cp, ri, va = (np.array(a) for a in oracle.csc(*shape, K))
    X = x.reshape(-1, batch)
    for col in (n + 2, (m // 2) * n + n // 2, (m // 2) * n + n // 2 + 1, (m - 1) * n + n - 2, (m // 3) * n + 63, (m // 3) * n + 64):
        X[col] = np.inf
        ri[cp[col]:cp[col + 1]] = np.arange(cp[col + 1] - cp[col]) + (3 * col) % (plan.cols - 200)
    plan.col_idx.copy_(torch.from_numpy(ri.astype(np.int32)))
    y = cs.conv_spmv_from_csc(plan, torch.from_numpy(X.reshape(-1)).to(device()), batch=batch)
    torch.cuda.synchronize()
    T = sp.csc_matrix((va.astype(np.float64), ri, cp), shape=(plan.cols, plan.rows))
    finite = np.isfinite(T @ np.where(np.isinf(X), np.inf, 0.0).astype(np.float64))
    got = y.cpu().numpy().reshape(-1, batch)
    assert np.array_equal(np.isfinite(got), finite) and not finite.all()
    X0 = np.where(np.isinf(X), 0.0, X).astype(np.float64)
    assert np.all(np.abs(got - T @ X0)[finite] <= (REL_TOL * (abs(T) @ np.abs(X0)) + 1e-30)[finite])
    plan.close()


def test_replays_follow_arrays_edited_between_them():
    """A captured product, replayed on arrays as built, edited, and as built again."""
    import scipy.sparse as sp
    shape, batch = (120, 133, 5, 1, 2), 9
    x, K = inputs(shape, batch, 13)
    plan = plan_of(shape, K, batch)
    cp, ri, va = (np.array(a) for a in oracle.csc(*shape, K))
    xd = torch.from_numpy(x).to(device())
    y = torch.empty(plan.cols * batch, device=device())
    cs.conv_spmv_from_csc(plan, xd, y, batch=batch)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cs.conv_spmv_from_csc(plan, xd, y, batch=batch)
    e = int(cp[61 * 133 + 40])
    for rep in range(6):
        rows = ri.copy()
        if rep in (1, 2, 4):
            rows[e + rep] = 7 * rep
        plan.col_idx.copy_(torch.from_numpy(rows.astype(np.int32)))
        y.fill_(float("nan"))
        graph.replay()
        eager = cs.conv_spmv_from_csc(plan, xd, batch=batch)
        torch.cuda.synchronize()
        T = sp.csc_matrix((va.astype(np.float64), rows, cp), shape=(plan.cols, plan.rows))
        X = x.reshape(-1, batch).astype(np.float64)
        want, scale = T @ X, abs(T) @ np.abs(X)
        for got in (y, eager):
            assert np.all(np.abs(got.cpu().numpy().reshape(-1, batch) - want) <= REL_TOL * scale + 1e-30), rep
    plan.close()


@pytest.mark.parametrize("shape,batch", [((24, 9100, 7, 1, 3), 128), ((30, 5000, 11, 1, 5), 64)])
def test_workgroups_that_start_while_the_plan_is_noted(shape, batch):
    """More workgroups than run at once, every column edited: the later ones read the note of the earlier ones while it is
    written, each as a whole."""
    x, K = inputs(shape, batch, 16)
    xd = torch.from_numpy(x).to(device())
    ref, scale = oracle.conv(*shape, x, K, batch=batch, want_scale=True)
    assert cs.conv_dispatch_info(*shape, batch, 3).kernel == 11 and cs.conv_dispatch_info(*shape, batch, 3).workgroups > 600
    for rep in range(3):
        plan = build_plan_t(shape, K)
        first = plan.row_ptr[:-1].long()
        first = first[plan.row_ptr[1:].long() - first > 1]           # the first two entries of a column change places
        for a in (plan.col_idx, plan.vals):
            b = a[first].clone()
            a[first] = a[first + 1]
            a[first + 1] = b
        y = torch.full((plan.cols * batch,), float("nan"), device=device())
        cs.conv_spmv_from_csc(plan, xd, y, batch=batch)
        got = y.cpu().numpy()
        assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= REL_TOL * scale), rep
        plan.close()


def test_a_plan_edited_on_two_streams_at_once():
    """Products of one edited plan side by side on two streams, of two batches (two launch shapes), first calls included."""
    import scipy.sparse as sp
    shape = (300, 260, 7, 1, 3)
    x, K = inputs(shape, 16, 14)
    cp, ri, va = (np.array(a) for a in oracle.csc(*shape, K))
    ri[int(cp[150 * 260 + 99]) + 3] = 5
    T = sp.csc_matrix((va.astype(np.float64), ri, cp), shape=(300 * 260, 300 * 260))
    xs = {b: torch.from_numpy(x[:300 * 260 * b]).to(device()) for b in (5, 16)}
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for rep in range(8):
        plan = plan_of(shape, K, 16)
        plan.col_idx.copy_(torch.from_numpy(ri.astype(np.int32)))
        ys = [torch.full((plan.cols * b,), float("nan"), device=device()) for b in (5, 16, 5, 16)]
        torch.cuda.synchronize()
        for i, y in enumerate(ys):
            b = y.numel() // plan.cols
            cs.conv_spmv_from_csc(plan, xs[b], y, batch=b, stream=streams[(i + rep) % 2])
        torch.cuda.synchronize()
        for y in ys:
            b = y.numel() // plan.cols
            X = xs[b].cpu().numpy().reshape(-1, b).astype(np.float64)
            assert np.all(np.abs(y.cpu().numpy().reshape(-1, b) - T @ X) <= REL_TOL * (abs(T) @ np.abs(X)) + 1e-30), (rep, b)
        plan.close()


def test_more_plans_than_places_for_the_note():
    """65536 plans at a time have a word to note edited columns in; one more scatters, and once the others are gone a plan takes the
    place of an earlier one, whose note it does not inherit."""
    import ctypes
    from paper_2411_19419_amd import binding
    lib, small = binding._load(), (3, 3, 2, 1, 1)
    arrays = build_plan_t(small, np.ones(4, dtype=np.float32))
    K4 = torch.ones(4, device=device())
    at = [t.data_ptr() for t in (K4, arrays.row_ptr, arrays.col_idx, arrays.vals)]
    handles = []
    for _ in range(65536):
        handle = ctypes.c_void_p()
        assert lib.conv_csc_build(*small, *at, None, ctypes.byref(handle)) == 0
        handles.append(handle)
    shape, batch = (90, 129, 3, 1, 1), 18
    x, K = inputs(shape, batch, 17)
    ref, scale = oracle.conv(*shape, x, K, batch=batch, want_scale=True)
    xd = torch.from_numpy(x).to(device())

    def product(edited):
        plan = plan_of(shape, K, batch)
        if edited:                                                   # the first two entries of a column change places
            e = int(plan.row_ptr[700])
            for a in (plan.col_idx, plan.vals):
                a[e:e + 2] = a[e:e + 2].flip(0)
        for _ in range(2):
            got = cs.conv_spmv_from_csc(plan, xd, batch=batch).cpu().numpy()
            assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= REL_TOL * scale)
        plan.close()
    product(False)
    product(True)
    torch.cuda.synchronize()
    for handle in handles:
        assert lib.conv_plan_destroy(handle) == 0
    for edited in (True, False, True):
        product(edited)
    arrays.close()
