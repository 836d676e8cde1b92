"""Merges of many short split lines: a lane group per line (up to 8 chunks), with lines for the
wave (up to 32) and for the block among them, at the number of lines from which lane groups
take lines of their own and one below, and a last block of fewer lines."""
import numpy as np
import pytest
import torch

import oracle
import paper_2203_07673_amd as F
from tests.gat_gate import gat_backward_magnitudes, kink_free
from tests.gates import TOL_F32, TOL_F64
from tests.gpu_helpers import dev, gate, host, log, ref_fusedmm_a
from workloads import CsrPattern, dense_normal

pytestmark = pytest.mark.gpu

CHUNK = 2
LANES = {(4, 4): 1, (8, 4): 2, (13, 1): 16, (16, 4): 4, (60, 4): 16, (2, 2): 1, (32, 2): 16}


def _pattern(n_splits, npdt):
    """Split lines of two to four chunks, some of 7, 8, 9, 31, 32, 33 and 65, and whole lines between."""
    rng = np.random.default_rng(841)
    chunks = rng.integers(2, 5, n_splits)
    at = rng.choice(n_splits, 70, replace=False)
    chunks[at] = np.resize([7, 8, 9, 31, 32, 33, 65], 70)
    chunks[-1] = 8
    lens = np.stack([rng.integers(0, CHUNK + 1, n_splits), CHUNK * chunks - rng.integers(0, 2, n_splits)], 1).reshape(-1)
    n = lens.size
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    first = rng.integers(0, n - 3 * lens.max(), n)
    pos = np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lens)
    cols = np.repeat(first, lens) + pos * 3 - (pos % 2)  # ascending
    return CsrPattern(n, n, rowptr, cols.astype(np.int32), rng.random(rowptr[-1]).astype(npdt))


CASES = [(r, np.float32, d) for r in (4, 8, 13, 16, 60) for d in (-1, 0, 5)] + [(r, np.float64, 3) for r in (2, 32)]


@pytest.mark.parametrize("r,npdt,d", CASES)
def test_packed_line_merges(r, npdt, d):
    vw = (4 if npdt == np.float32 else 2) if r != 13 else 1
    n_splits = 1024 * (64 // LANES[r, vw]) + d
    S = _pattern(n_splits, npdt)
    tol = TOL_F64 if npdt == np.float64 else TOL_F32
    A, B, C0 = (dense_normal(S.m, r, 842 + k, dtype=npdt) for k in range(3))
    log(f"packed merges r={r} {npdt.__name__} splits={n_splits}")
    P = F.Pattern.from_csr(S, long_len=CHUNK, chunk=CHUNK)
    assert P.schedules["csr"]["n_splits"] == n_splits
    ref, mag = ref_fusedmm_a(S, A, B)
    big = torch.full((S.m * r + 8,), 7.0, dtype=torch.float64 if npdt == np.float64 else torch.float32, device="cuda")
    out = big[4:-4].view(S.m, r)
    F.fusedmm_a_raw(P, dev(A), dev(B), out=out)
    gate("C", host(out), ref, mag, tol)
    assert bool((big[:4] == 7).all()) and bool((big[-4:] == 7).all())
    out = dev(C0).clone()
    F.spmm_a_raw(P, dev(B), out=out, beta=-0.5)
    gate("SB", host(out), -0.5 * C0 + oracle.spmm_a(S, S.val, B),
         0.5 * np.abs(C0) + oracle.spmm_a(S, S.val, np.abs(B)), tol)


@pytest.mark.parametrize("r,lanes", [(8, 2), (16, 4)])
def test_packed_bf16_gradients(r, lanes):
    """The merge that rounds to bfloat16: the bits of the float32 merge rounded."""
    from paper_2203_07673_amd import fusedmm as M
    S = _pattern(1024 * (64 // lanes) + 7, np.float32)
    log(f"packed bf16 merges r={r}")
    P = F.Pattern.from_csr(S, long_len=CHUNK, chunk=CHUNK)
    A, B = (F.to_bf16(dev(dense_normal(S.m, r, 851 + k))) for k in (0, 1))
    G = dev(dense_normal(S.m, r, 853))
    want = M._fused_backward("a", P, A, B, G, None, None, (True, True), True, None, None)
    got = M._fused_backward("a", P, A, B, G, None, None, (True, True), True, None, None, True)
    for g, w in zip(got, want):
        assert torch.equal(g, w.to(torch.bfloat16))


@pytest.mark.parametrize("r,lanes", [(16, 4), (60, 16)])
def test_packed_attention_merges(r, lanes):
    S = _pattern(1024 * (64 // lanes) + 9, np.float32)
    H, dO = dense_normal(S.n, r, 861), dense_normal(S.m, r, 864)
    a1, a2 = (dense_normal(1, r, 862 + k, sigma=r ** -0.5)[0] for k in (0, 1))
    S, _ = kink_free(S, H, a1, a2)
    log(f"packed attention merges r={r}")
    P = F.Pattern.from_csr(S, long_len=CHUNK, chunk=CHUNK)
    s, t = oracle.gat_scores(H, a1, a2)
    ms, mt = oracle.gat_scores(np.abs(H), np.abs(a1), np.abs(a2))
    rows = np.repeat(np.arange(S.m), np.diff(S.rowptr))
    for softmax in (True, False):
        w = oracle.gat_edges(S, s, t, 0.2, softmax)
        size = S.val * (ms[rows] + mt[S.colidx])  # rounding of a score, in units of u
        if softmax:  # moves its weight, and the row's sum, by as much
            top = np.zeros(S.m)
            np.maximum.at(top, rows, size)
            size = w * (1 + size + top[rows])
        out = F.gat_forward(P, dev(H), dev(a1), dev(a2), softmax=softmax)
        gate("out", host(out), oracle.spmm_a(S, w, H), oracle.spmm_a(S, size, np.abs(H)), TOL_F32)
        want = oracle.gat_backward(S, H, a1, a2, dO, slope=0.2, softmax=softmax)
        sizes = gat_backward_magnitudes(S, H, a1, a2, dO, slope=0.2, softmax=softmax)
        for name, g, x, m in zip(("dH", "da1", "da2", "dS"),
                                 F.gat_backward(P, dev(H), dev(a1), dev(a2), out, dev(dO), softmax=softmax, want_dS=True),
                                 want, sizes):
            gate(name, host(g), x, m, TOL_F32)
