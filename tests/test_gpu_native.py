"""The repeated calls through the native module against the same calls through ctypes: results, what is refused and how,
streams, and plans that are closed or dropped."""
import threading

import numpy as np
import pytest
import torch

import paper_2411_19419_amd as cs
from gpu_util import device
from paper_2411_19419_amd import binding

pytestmark = pytest.mark.gpu


def _both(monkeypatch, call):
    """What a call returns, or raises, with the native module and without it."""
    got = []
    for native in (binding._native, None):
        with monkeypatch.context() as patch:
            if native is None:
                patch.setattr(binding, "_native", None)
            try:
                got.append(call())
            except Exception as e:
                got.append((type(e), str(e)))
    return got


def test_results_and_refusals_are_alike(monkeypatch):
    torch.manual_seed(0)
    shape, batch = (21, 18, 3, 2, 1), 5
    K = torch.randn(9, device=device())
    plan, plan_t = cs.conv_csr_build(*shape, K), cs.conv_csc_build(*shape, K)
    assert binding._native is not None
    x, y = torch.randn(plan.cols * batch, device=device()), torch.empty(plan.rows * batch, device=device())
    z = torch.empty(plan.cols * batch, device=device())
    pitched = torch.empty(2 * y.numel(), device=device())[::2]
    overlap = torch.empty(x.numel() + y.numel(), device=device())

    class Own(torch.Tensor):
        pass

    calls = [lambda: cs.conv_spmv(plan, x, y, batch=batch).clone(), lambda: cs.conv_spmv(plan_t, y, z, batch=batch).clone(),
             lambda: cs.conv_spmv_from_csc(plan_t, x, y, batch=batch).clone(), lambda: cs.conv_spmv(plan, x, batch=batch).clone(),
             lambda: cs.conv_spmv(plan, x.as_subclass(Own), y, batch=batch).clone().as_subclass(torch.Tensor),
             lambda: cs.conv_spmv(plan, x, y, batch=np.int64(batch)).clone(),
             lambda: cs.conv_spmv(plan, x.double(), y, batch=batch), lambda: cs.conv_spmv(plan, x, pitched, batch=batch),
             lambda: cs.conv_spmv(plan, x.cpu(), y, batch=batch), lambda: cs.conv_spmv(plan, x, y, batch=batch + 1),
             lambda: cs.conv_spmv(plan, x, y, batch=0), lambda: cs.conv_spmv(plan, x, y, batch=-1), lambda: cs.conv_spmv(plan, None, y, batch=batch),
             lambda: cs.conv_spmv(plan, overlap[:x.numel()], overlap[x.numel() - 3:x.numel() - 3 + y.numel()], batch=batch),
             lambda: cs.conv_spmv_from_csc(plan, x, y, batch=batch), lambda: cs.conv_spmv_from_csc(plan, y, x, batch=batch),
             lambda: cs.conv_update_kernel(plan, K[:8]), lambda: cs.conv_update_kernel(plan, K.cpu()), lambda: cs.conv_update_kernel(plan, 2 * K)]
    for i, call in enumerate(calls):
        native, plain = _both(monkeypatch, call)
        assert type(native) is type(plain), (i, native, plain)
        if i == 2:        # (a scatter, whose adds arrive in any order: up to four per output, of a few units each)
            assert torch.allclose(native, plain, rtol=1e-6, atol=1e-5)
        else:
            assert torch.equal(native, plain) if isinstance(native, torch.Tensor) else native == plain, (i, native, plain)
    for build in (cs.conv_csr_build, cs.conv_csc_build):
        for args in (shape, (5, 4, 3, 1, 7), (3, 3, 1, 1, 0), (2, 2, 1, 4, 3), (4, 4, 9, 1, 0), (0, 4, 1, 1, 0), (4, 4, 3, 0, 0), (4, 4, 3, 1, -1),
                     (4.0, 4, 3, 1, 1), (70000, 70000, 3, 1, 1)):
            native, plain = _both(monkeypatch, lambda: build(*args, torch.ones(int(args[2]) ** 2, device=device())))
            if isinstance(native, tuple):
                assert native == plain, args
                continue
            for name in ("m_out", "n_out", "nnz", "rows", "cols", "transposed", "_home", "_elsewhere"):
                assert getattr(native, name) == getattr(plain, name), (args, name)
            for a, b in ((native.row_ptr, plain.row_ptr), (native.col_idx, plain.col_idx), (native.vals, plain.vals)):
                assert torch.equal(a, b) and a.dtype == b.dtype and a.is_contiguous(), args
    for pl in (plan, plan_t):
        pl.close()
        pl.close()
    native, plain = _both(monkeypatch, lambda: cs.conv_spmv(plan, x, y, batch=batch))
    assert native == plain and native[0] is ValueError


def test_streams_and_threads():
    """Each thread's current stream is the one that is used, and the plan knows that another stream has seen it."""
    shape = (40, 41, 3, 1, 1)
    plan = cs.conv_csr_build(*shape, torch.randn(9, device=device()))
    x = torch.randn(plan.cols, device=device())
    want = cs.conv_spmv(plan, x, torch.empty(plan.rows, device=device()))
    assert not plan._elsewhere
    torch.cuda.synchronize()
    got = [None] * 4

    def work(i):
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            y = torch.empty(plan.rows, device=device())
            for _ in range(50):
                cs.conv_spmv(plan, x, y)
        side.synchronize()
        got[i] = y

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert plan._elsewhere and all(torch.equal(y, want) for y in got)
    plan.close()
