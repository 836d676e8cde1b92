"""The order of the sums of batched CG: one for every kernel of a solve, and in float32 that of a
pass over the lines per iteration, also for rows of over 64 elements in no whole vectors.  A
solve goes on after short lines have converged, on quotients of rounding errors, so another
order shows in the result."""
import numpy as np
import pytest
import torch

import oracle
import paper_2203_07673_amd as F
from paper_2203_07673_amd import _capi as C
from tests.gpu_helpers import dev, host, log
from tests.test_gpu_als import _fma, _rows_sum, _tree
from workloads import CsrPattern, dense_normal

pytestmark = pytest.mark.gpu


def _dot(y, z):
    """Elements 64 apart in a chain, then a tree over the 64 lanes."""
    y, z = (np.concatenate([x, np.zeros(-len(x) % 64, np.float32)]).reshape(-1, 64) for x in (y, z))
    s = y[0] * z[0]
    for a, b in zip(y[1:], z[1:]):
        s = _fma(a, b, s)
    return _tree(s)


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("r", [65, 99, 127, 129, 130, 193, 255])
def test_wide_rows_of_no_whole_vectors(r, split):
    lens = (0, 1, 7, 8, 9, 36, 37, 48, 49, 72, 73, 90, 110)
    rng = np.random.default_rng(881)
    n, lam, iters = 150, np.float32(0.05), 4
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cols = np.concatenate([np.sort(rng.choice(n, k, replace=False)) for k in lens]).astype(np.int32)
    val = rng.standard_normal(rowptr[-1]).astype(np.float32)
    S = CsrPattern(len(lens), n, rowptr, cols, val)
    Fa, X = dense_normal(n, r, 882, sigma=r ** -0.5), dense_normal(len(lens), r, 883)
    log(f"cg order of wide rows r={r} split={split}")
    P = F.Pattern.from_csr(S, split=split, long_len=80, chunk=30)
    want = X.copy()
    for i in range(len(lens)):
        js, v = Fa[cols[rowptr[i]:rowptr[i + 1]]], val[rowptr[i]:rowptr[i + 1]]
        chunk = 30 if split and len(v) > 80 else n

        def gram(y):
            return _fma(y, lam, _rows_sum(np.array([_dot(y, f) for f in js], np.float32), js, chunk))

        x = want[i]
        res = _rows_sum(v, js, chunk) - gram(x)
        p, rr = res, _dot(res, res)
        for _ in range(iters):
            q = gram(p)
            pq = _dot(p, q)
            alpha = rr / pq if rr > 0 and pq > 0 else np.float32(0)
            x, res = _fma(p, alpha, x), _fma(q, -alpha, res)
            new = _dot(res, res)
            p, rr = _fma(p, new / rr if rr > 0 else np.float32(0), res), new
        want[i] = x
    Xd = dev(X).clone()
    F.fusedmm._als_lines(P, C.FMM_CSR, dev(Fa), float(lam), iters, Xd)
    assert np.array_equal(host(Xd).astype(np.float32), want)


@pytest.mark.parametrize("r,dtype", [(r, torch.float32) for r in (1, 3, 5, 50, 63, 64, 65, 99, 130, 255, 256, 516, 1024)] +
                         [(r, torch.bfloat16) for r in (8, 24, 64, 72, 136, 256, 264, 512, 520, 1024)])
def test_split_lines_sum_like_whole_ones(r, dtype):
    """Lines whose last entry, a chunk of its own where they are split, gathers zeros: the solve
    of split lines has the bits of the solve in one kernel."""
    rng = np.random.default_rng(891)
    n, chunk = 60, 20
    lens = np.array([chunk + 1, 3, chunk + 1, chunk + 1])
    cols = np.concatenate([np.append(np.sort(rng.choice(n - 1, k - 1, replace=False)), n - 1) for k in lens]).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    S = CsrPattern(len(lens), n, rowptr, cols, rng.standard_normal(rowptr[-1]).astype(np.float32))
    Fa = dense_normal(n, r, 892, sigma=r ** -0.5)
    Fa[n - 1] = 0
    Fd = dev(oracle.bf16_round(Fa) if dtype == torch.bfloat16 else Fa, dtype)
    X0, rhs = dev(dense_normal(len(lens), r, 893)), dev(dense_normal(len(lens), r, 894))
    log(f"split like whole r={r} {dtype}")
    got = []
    for split in (False, True):
        P = F.Pattern.from_csr(S, split=split, long_len=chunk, chunk=chunk)
        assert bool(P.schedules["csr"]) == split
        X, Y = X0.clone(), X0.clone()
        F.cg_lines(P, C.FMM_CSR, Fd, rhs, 0.25, 6, X)
        F.fusedmm._als_lines(P, C.FMM_CSR, Fd, 0.25, 6, Y)
        got.append((X, Y))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
