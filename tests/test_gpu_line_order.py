"""A line order that the caller gives is the one the passes follow; only the default that
Pattern sets by itself is left out, for fused passes over wide rows of many lines."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2203_07673_amd as F
from paper_2203_07673_amd import _capi as C
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


def _pattern(m, n, **kw):
    """Lines of one entry and one of ten, so that the default orders them."""
    lens = np.ones(m, np.int64)
    lens[5] = 10
    ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    idx = (np.arange(ptr[-1]) % n).astype(np.int32)
    idx[ptr[5]:ptr[6]] = np.arange(10)
    return F.Pattern(ptr, idx, None, (m, n), **kw)


@pytest.mark.parametrize("r,dtype", [(256, torch.float32), (512, torch.bfloat16)])
def test_given_order_is_followed(r, dtype):
    """An order that names the even lines twice: the odd lines keep what the output held."""
    log(f"given order r={r} {dtype}")
    m, n = 1 << 18, 16
    P = _pattern(m, n, line_order=False)
    A, B = torch.ones(m, r, device="cuda", dtype=dtype), torch.ones(n, r, device="cuda", dtype=dtype)
    order = torch.arange(m, device="cuda", dtype=torch.int32) // 2 * 2
    d = P.descriptor(C.FMM_CSR)
    d.order = order.data_ptr()
    out = torch.full((m, r), -7.0, device="cuda")
    torch.cuda.synchronize()
    C.call("fmm_fusedmm_a", ctypes.byref(d), A.data_ptr(), B.data_ptr(), r, F.dtype_code(A), out.data_ptr(), C.FMM_FUSED,
           None, None, 0, torch.cuda.current_stream().cuda_stream)
    assert bool((out[1::2] == -7.0).all()) and bool((out[0::2] == r).all())


def test_only_the_default_order_is_left_out():
    log("default order")
    m, n = 1 << 18, 16
    P = _pattern(m, n)
    X = {(r, t): torch.empty(0, r, device="cuda", dtype=t)
         for r in (128, 252, 256, 512) for t in (torch.float32, torch.bfloat16, torch.float64)}

    def ordered(P, r, t, two=False):
        return bool(P._fused_desc(C.FMM_CSR, two, X[r, t]).order)

    assert P.orders["csr"] is not None
    for r, t, want in ((128, torch.float32, True), (252, torch.float32, True), (256, torch.float32, False),
                       (256, torch.bfloat16, True), (512, torch.bfloat16, False), (512, torch.float64, True)):
        assert ordered(P, r, t) == want, (r, t)
    assert ordered(P, 128, torch.float32, two=True)  # 512-byte rows: from 2^20 lines
    Q = P.with_values(torch.ones(P.nnz, device="cuda"))
    P.set_line_order(C.FMM_CSR, True)
    assert ordered(P, 256, torch.float32) and not ordered(Q, 256, torch.float32)
    for R in (_pattern(m, n, line_order=True), _pattern(m - 1, n)):
        assert ordered(R, 256, torch.float32)
    R = _pattern(1 << 20, n)
    assert not ordered(R, 128, torch.float32, two=True) and ordered(R, 128, torch.float32)
    t = P.tuning
    R = _pattern(m, n)
    R.apply_tuning(t)
    assert R.tuning == t and ordered(R, 256, torch.float32)


def test_index_order_under_capture():
    """Going back to index order asks nothing of the GPU, so a program may do it while it
    captures a graph."""
    log("index order under capture")
    P = _pattern(3000, 16, line_order=True)
    A, B, out = torch.randn(3000, 64, device="cuda"), torch.randn(16, 64, device="cuda"), torch.empty(3000, 64, device="cuda")
    want = F.fusedmm_a_raw(P, A, B)[0]
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        P.set_line_order(C.FMM_CSR, False)
        F.fusedmm_a_raw(P, A, B, out=out)
    assert P.orders["csr"] is None
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
