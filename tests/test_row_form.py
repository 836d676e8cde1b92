"""Rows whose length is no multiple of the vector: which passes take them in overlapping
vectors and which by elements, and the results of the passes by elements."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2203_07673_amd as F
from paper_2203_07673_amd import _capi as C
from tests.gates import TOL_F32
from tests.gpu_helpers import (dev, gate, host, log, ref_fusedmm_a, ref_fusedmm_a_backward, ref_fusedmm_b_backward,
                               ref_sddmm)
from workloads import CsrPattern, dense_normal


def _form(r, lines, minor, mean, two_row, dtype=C.FMM_F32, n_chunks=0):
    """(lanes, elements per vector) of a pass over lines of a `lines` x `minor` pattern."""
    d = C.fmm_sparse()
    d.orient, d.rows, d.cols, d.nnz = C.FMM_CSR, lines, minor, lines * mean
    d.ptr = d.idx = 16
    if n_chunks:
        d.chunks = d.splits = 16
        d.long_len, d.n_chunks, d.n_splits = 128, n_chunks, 1
    out = [ctypes.c_int32(0) for _ in range(4)]
    assert C.load().fmm_launch_shape(ctypes.byref(d), int(two_row), r, dtype, *[ctypes.byref(x) for x in out]) == 0
    return out[0].value, out[2].value


@pytest.mark.parametrize("two_row,r,lines,mean,lanes,vw", [
    # one row gathered: by elements for 17 to 32 of them, lines of 12 and more, past 12 MB
    (False, 27, 300000, 30, 32, 1), (False, 21, 300000, 30, 32, 1), (False, 27, 131072, 16, 32, 1),
    (False, 33, 300000, 30, 16, 4), (False, 21, 131072, 16, 8, 4), (False, 27, 262144, 8, 8, 4),
    (False, 61, 300000, 30, 16, 4), (False, 28, 300000, 30, 8, 4), (False, 13, 300000, 30, 16, 1),
    # two rows: 17 to 32 past 8 MB, 33 to 64 between 48 and 400 MB
    (True, 27, 300000, 30, 32, 1), (True, 17, 131072, 16, 32, 1), (True, 27, 262144, 8, 32, 1),
    (True, 25, 32768, 16, 8, 4), (True, 38, 300000, 30, 64, 1), (True, 61, 131072, 16, 64, 1),
    (True, 38, 131072, 16, 16, 4), (True, 46, 262144, 8, 16, 4), (True, 50, 1 << 20, 16, 16, 4),
    (True, 75, 300000, 30, 32, 4), (True, 60, 300000, 30, 16, 4)])
def test_row_form(two_row, r, lines, mean, lanes, vw):
    assert _form(r, lines, lines, mean, two_row) == (lanes, vw)
    # a power-law pattern has split lines: in vectors, a small one by elements
    small = r <= 64 and lines * mean * (64 if r > 32 else 32) <= (1 << 25 if two_row else 1 << 24) and r % 4
    assert _form(r, lines, lines, mean, two_row, n_chunks=100)[1] == (1 if r <= 16 or small else 4)
    # nothing but float32 goes by elements above 16 of them
    assert _form(r, lines, lines, mean, two_row, C.FMM_F64)[1] == 2


@pytest.mark.parametrize("two_row", [False, True])
@pytest.mark.parametrize("r,lanes", [(17, 32), (31, 32), (33, 64), (63, 64)])
def test_row_form_of_small_split_patterns(two_row, r, lanes):
    """Split lines: by elements while entries times lanes stay below 2^24 (one row), 2^25 (two)."""
    limit = (1 << 25 if two_row else 1 << 24) // lanes // 8  # lines of 8 entries
    assert _form(r, limit, 1000, 8, two_row, n_chunks=3) == (lanes, 1)
    assert _form(r, limit + 1, 1000, 8, two_row, n_chunks=3) == (8 if r <= 32 else 16, 4)
    assert _form(r, 100, 1000, 8, two_row, C.FMM_F64, n_chunks=3)[1] == 2
    assert _form(r + 64, 100, 1000, 8, two_row, n_chunks=3)[1] == 4


def test_given_shape_is_taken():
    lib = C.load()
    try:
        assert lib.fmm_set_tuning(64, 1) == 0
        assert _form(27, 300000, 300000, 30, False) == (64, 4)
    finally:
        assert lib.fmm_set_tuning(0, 0) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("r", [17, 21, 31, 33, 50, 63])
def test_rows_by_elements(r):
    """300 lines over a wide matrix, whose passes over rows take the rows by elements: every
    operation against the oracle, on bases aligned to one element, between guards."""
    log(f"rows by elements r={r}")
    m, n, deg = 300, 260000, 13
    rng = np.random.default_rng(31)
    lens = np.full(m, deg)
    lens[3], lens[4], lens[7] = 0, 1, 100
    cols = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lens]).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    S = CsrPattern(m, n, rowptr, cols, rng.random(rowptr[-1]).astype(np.float32))
    P = F.Pattern.from_csr(S)
    one, two = (P.launch_shape(C.FMM_CSR, t, r, C.FMM_F32)[2] for t in (False, True))
    assert two == 1 and one == (1 if r <= 32 else 4)
    A, B = dense_normal(m, r, 32), dense_normal(n, r, 33)
    G, Gb = dense_normal(m, r, 34), dense_normal(n, r, 35)

    def shifted(x):
        big = torch.zeros(x.size + 1, device="cuda")
        big[1:] = dev(x.reshape(-1))
        return big[1:].view(*x.shape)

    Ad, Bd, Gd, Gbd = shifted(A), shifted(B), shifted(G), shifted(Gb)
    big = torch.full((m * r + 10,), 7.0, device="cuda")
    out = big[5:5 + m * r].view(m, r)
    ref, mag = ref_fusedmm_a(S, A, B)
    for fused in (True, False):
        F.fusedmm_a_raw(P, Ad, Bd, out=out, fused=fused)
        gate("C", host(out), ref, mag, TOL_F32)
    assert bool((big[:5] == 7).all()) and bool((big[-5:] == 7).all())
    ref, mag = ref_sddmm(S, A, B)
    gate("R", host(F.sddmm_raw(P, Ad, Bd)), ref, mag, TOL_F32)
    a = ref_fusedmm_a_backward(S, A, B, G)
    dS, gA = F.fusedmm_a_backward_values_raw(P, Ad, Bd, Gd, want_dA=True)
    gate("dA", host(gA), a[0], a[2], TOL_F32)
    Sa = oracle.absolute(S)
    gate("dS", host(dS), oracle.fusedmm_a_backward_values(S, A, B, G),
         oracle.fusedmm_a_backward_values(Sa, np.abs(A), np.abs(B), np.abs(G)), TOL_F32)
    b = ref_fusedmm_b_backward(S, A, B, Gb)
    for fused in (True, False):  # the transposed form's two-row pass runs on the rows
        R = None if fused else F.fusedmm_b_raw(P, Ad, Bd, fused=False)[1]
        gA, _ = F.fusedmm_b_backward_raw(P, Ad, Bd, Gbd, fused=fused, R_ws=R)
        gate("dA'", host(gA), b[0], b[2], TOL_F32)
    P.set_gather_hints(C.FMM_CSR, 5)
    assert torch.equal(F.fusedmm_b_backward_raw(P, Ad, Bd, Gbd)[0], F.fusedmm_b_backward_raw(F.Pattern.from_csr(S), Ad, Bd, Gbd)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("long_len", [128, 16])
@pytest.mark.parametrize("r", [17, 31, 33, 63])
def test_split_lines_by_elements(r, long_len):
    """A small pattern with split lines, whose passes go by elements: every operation in both
    orientations against the oracle, on bases aligned to one element."""
    log(f"split lines by elements r={r} long_len={long_len}")
    m, n = 260, 700
    rng = np.random.default_rng(41)
    lens = rng.integers(0, 12, m)
    lens[0], lens[5], lens[6], lens[259] = 700, 129, 128, 300
    cols = [np.sort(rng.choice(n, k, replace=False)) for k in lens]
    for i in range(20, 220):  # and one long column
        if 3 not in cols[i]:
            cols[i] = np.sort(np.append(cols[i], 3))
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    S = CsrPattern(m, n, rowptr, np.concatenate(cols).astype(np.int32), rng.random(rowptr[-1]).astype(np.float32))
    P = F.Pattern.from_csr(S, long_len=long_len, chunk=long_len)
    for orient in (C.FMM_CSR, C.FMM_CSC):
        assert P.splits["csr" if orient == C.FMM_CSR else "csc"] == long_len
        for two_row in (False, True):
            assert P.launch_shape(orient, two_row, r, C.FMM_F32)[2] == 1
    A, B = dense_normal(m, r, 42), dense_normal(n, r, 43)
    G, Gb = dense_normal(m, r, 44), dense_normal(n, r, 45)

    def shifted(x):
        big = torch.zeros(x.size + 1, device="cuda")
        big[1:] = dev(x.reshape(-1))
        return big[1:].view(*x.shape)

    Ad, Bd, Gd, Gbd = shifted(A), shifted(B), shifted(G), shifted(Gb)
    ref, mag = ref_sddmm(S, A, B)
    gate("R", host(F.sddmm_raw(P, Ad, Bd)), ref, mag, TOL_F32)
    ref, mag = ref_fusedmm_a(S, A, B)
    a = ref_fusedmm_a_backward(S, A, B, G)
    b = ref_fusedmm_b_backward(S, A, B, Gb)
    for fused in (True, False):
        out, R = F.fusedmm_a_raw(P, Ad, Bd, fused=fused)
        gate("C", host(out), ref, mag, TOL_F32)
        gA, gB = F.fusedmm_a_backward_raw(P, Ad, Bd, Gd, fused=fused, R_ws=R)
        gate("dA", host(gA), a[0], a[2], TOL_F32)
        gate("dB", host(gB), a[1], a[3], TOL_F32)
        R = None if fused else F.fusedmm_b_raw(P, Ad, Bd, fused=False)[1]
        gA, gB = F.fusedmm_b_backward_raw(P, Ad, Bd, Gbd, fused=fused, R_ws=R)
        gate("dA'", host(gA), b[0], b[2], TOL_F32)
        gate("dB'", host(gB), b[1], b[3], TOL_F32)
    dS, gA = F.fusedmm_a_backward_values_raw(P, Ad, Bd, Gd, want_dA=True)
    gate("dA", host(gA), a[0], a[2], TOL_F32)
    Sa = oracle.absolute(S)
    gate("dS", host(dS), oracle.fusedmm_a_backward_values(S, A, B, G),
         oracle.fusedmm_a_backward_values(Sa, np.abs(A), np.abs(B), np.abs(G)), TOL_F32)
