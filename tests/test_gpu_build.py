"""The fills where a workgroup walks down several lines, with rows of odd and of even length, and the
sweep of many products at batches in chunks: bit-exact arrays, products against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2411_19419_amd as cs
from gpu_util import REL_TOL, build_plan, build_plan_t, check_csc, check_csr, device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1500, 700, 3, 1, 1),      # two lines per workgroup (indices), five (values); T^T alike
    (2100, 900, 2, 2, 0),      # rows of four entries: gaps in the image; T^T rows of one
    (1300, 700, 4, 1, 2),      # rows of sixteen
    (2500, 600, 1, 3, 0),      # rows of one; lines of T^T without entries
    (1400, 520, 5, 3, 2),      # T^T: rows of one, two and four entries
    (2000, 300, 3, 1, 2),      # ragged lengths at both borders, the last range short
    (40, 5000, 6, 1, 5),       # few lines, many ranges
])
def test_fills_over_several_lines(shape):
    m, n, k, s, p = shape
    rng = np.random.default_rng(3)
    K = rng.standard_normal(k * k).astype(np.float32)
    plan, plan_t = build_plan(shape, K), build_plan_t(shape, K)
    check_csr(plan, shape, K)
    check_csc(plan_t, shape, K)
    K2 = rng.standard_normal(k * k).astype(np.float32)
    for pl in (plan, plan_t):
        pl.vals.fill_(float("nan"))
        cs.conv_update_kernel(pl, torch.from_numpy(K2).to(device()))
    torch.cuda.synchronize()
    check_csr(plan, shape, K2)
    check_csc(plan_t, shape, K2)
    plan.close()
    plan_t.close()


@pytest.mark.parametrize("shape,channels", [     # fewer than 2 M values and 100 000 rows: through an image in LDS, more: in place
    ((28, 28, 3, 1, 1), 1), ((31, 33, 4, 1, 2), 1), ((470, 471, 3, 1, 1), 1), ((473, 475, 3, 1, 1), 1), ((500, 401, 6, 2, 3), 1),
    ((97, 700, 6, 2, 3), 1), ((300, 301, 3, 1, 1), 1), ((350, 301, 3, 1, 1), 1), ((250, 180, 3, 1, 1), 2), ((300, 301, 3, 1, 1), 3), ((90, 40, 11, 1, 10), 1), ((200, 1, 1, 1, 0), 1),
])
def test_new_kernels_of_few_and_many_values(shape, channels):
    m, n, k, s, p = shape
    rng = np.random.default_rng(7)
    K, K2 = (rng.standard_normal(channels * k * k).astype(np.float32) for _ in range(2))
    Kd = torch.from_numpy(K).to(device())
    plan = cs.conv_csr_build_channels(*shape, Kd, channels) if channels > 1 else build_plan(shape, K)
    plan.vals.fill_(float("nan"))
    cs.conv_update_kernel(plan, torch.from_numpy(K2).to(device()))
    torch.cuda.synchronize()
    parts = K2.reshape(channels, k * k)
    assert np.array_equal(plan.vals.cpu().numpy(), np.concatenate([oracle.csr(*shape, w)[2] for w in parts]))
    plan.close()
    if channels == 1:
        plan_t = build_plan_t(shape, K)
        plan_t.vals.fill_(float("nan"))
        cs.conv_update_kernel(plan_t, torch.from_numpy(K2).to(device()))
        torch.cuda.synchronize()
        check_csc(plan_t, shape, K2)
        plan_t.close()


@pytest.mark.parametrize("batch", [2, 4, 5, 8, 11, 16, 21])
def test_sweep_at_batches_in_chunks(batch):
    rng = np.random.default_rng(batch)
    shapes = [(30, 41, 3, 1, 1), (17, 17, 7, 2, 3), (9, 50, 1, 1, 0), (25, 12, 5, 1, 2), (8, 8, 2, 2, 0)]
    plans, xs, ys, refs = [], [], [], []
    for m, n, k, s, p in shapes:
        K = rng.standard_normal(k * k).astype(np.float32)
        x = rng.standard_normal(m * n * batch).astype(np.float32)
        plans.append(build_plan((m, n, k, s, p), K))
        xs.append(torch.from_numpy(x).to(device()))
        ys.append(torch.full((plans[-1].rows * batch,), float("nan"), dtype=torch.float32, device=device()))
        refs.append(oracle.conv(m, n, k, s, p, x, K, batch=batch, want_scale=True))
    multi = cs.ConvMulti(plans, xs, ys, batch=batch)
    multi.apply()
    torch.cuda.synchronize()
    for y, (ref, scale) in zip(ys, refs):
        got = y.cpu().numpy()
        assert not np.any(np.isnan(got)) and np.all(np.abs(got.astype(np.float64) - ref) <= REL_TOL * scale)
    multi.close()
    for pl in plans:
        pl.close()


SPIN = 20_000_000       # clock ticks of a waiting kernel: milliseconds, while the host goes on


def test_a_dropped_plan_waits_for_work_on_another_stream():
    """close() leaves the device alone when the plan was used on the default stream only, and waits for
    it when it was used on another (its arrays could be handed out again while they are read)."""
    K = torch.ones(9, device=device())
    plan = cs.conv_csr_build(64, 64, 3, 1, 1, K)
    x = torch.ones(64 * 64, device=device())
    cs.conv_spmv(plan, x)
    assert not plan._elsewhere
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    y = torch.empty(plan.rows, device=device())
    with torch.cuda.stream(side):
        torch.cuda._sleep(SPIN)
    cs.conv_spmv(plan, x, y, stream=side)
    assert plan._elsewhere and not side.query()
    plan.close()
    assert side.query()


@pytest.mark.parametrize("how", ["built", "replayed"])
def test_a_dropped_plan_of_a_side_stream_waits(how):
    """A plan built on a side stream reads a kernel that another stream's pool may get back, and a graph
    captured on that stream runs wherever it is replayed: close() waits for both."""
    K = torch.ones(9, device=device())
    x, y = torch.ones(64 * 64, device=device()), torch.empty(64 * 64, device=device())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        if how == "built":
            torch.cuda._sleep(SPIN)
        plan = cs.conv_csr_build(64, 64, 3, 1, 1, K)
    busy = side
    if how == "replayed":
        cs.conv_spmv(plan, x, y, stream=side)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            cs.conv_spmv(plan, x, y)
        torch.cuda.synchronize()
        busy = torch.cuda.current_stream()
        torch.cuda._sleep(SPIN)
        graph.replay()
    assert not busy.query()
    plan.close()
    assert busy.query()


def test_a_kernel_of_another_streams_pool_outlives_the_build():
    """Built on the default stream from a kernel that was allocated on another: its memory is not handed
    out again before the build has read it, though the plan and the kernel are dropped at once."""
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        K = torch.ones(9, device=device())
    torch.cuda.synchronize()
    place = K.data_ptr()
    torch.cuda._sleep(SPIN)
    plan = cs.conv_csr_build(64, 64, 3, 1, 1, K)
    plan.close()
    del plan, K
    with torch.cuda.stream(side):
        again = torch.empty(9, device=device())
        reused = again.data_ptr() == place
    assert torch.cuda.default_stream().query() or not reused
