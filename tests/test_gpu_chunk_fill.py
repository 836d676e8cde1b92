"""Chunks of split lines by a wave each: not for one-row passes over short chunks.  Which kernel
ran shows in the bits, since the groups of a wave add their sums in another order."""
import numpy as np
import pytest
import torch

import paper_2203_07673_amd as F
from tests.gpu_helpers import dev, log
from workloads import dense_normal

pytestmark = pytest.mark.gpu


def _pattern(m, n, deg):
    rng = np.random.default_rng(871)
    first = rng.integers(0, n - deg, m)
    cols = (first[:, None] + np.arange(deg)[None, :]).astype(np.int32).reshape(-1)
    val = rng.random(m * deg).astype(np.float32)
    keep = slice(0, 64 * deg)  # the first lines as a pattern of their own, of few chunks
    ptr = (np.arange(m + 1) * deg).astype(np.int32)
    return F.Pattern(ptr, cols, val, (m, n)), F.Pattern(ptr[:65], cols[keep], val[keep], (64, n))


@pytest.mark.parametrize("r,dtype", [(8, torch.float32), (16, torch.float32), (32, torch.float32),
                                     (8, torch.bfloat16), (16, torch.bfloat16), (64, torch.bfloat16)])
@pytest.mark.parametrize("extra", [-1, 0, 40])
def test_short_chunks_by_groups(r, dtype, extra):
    """2^14 chunks and around, lines of 130: chunks of 128 and 2."""
    log(f"short chunks r={r} {dtype} {extra}")
    m, n = (1 << 13) + extra, 4000
    P, few = _pattern(m, n, 130)
    assert P.schedules["csr"]["n_chunks"] == 2 * m and few.schedules["csr"]["n_chunks"] == 128
    A, B, G = dev(dense_normal(m, r, 872)).to(dtype), dev(dense_normal(n, r, 873)).to(dtype), dev(dense_normal(m, r, 874))
    for fn in (lambda P, k: F.fusedmm_a_raw(P, A[:k], B)[0], lambda P, k: F.spmm_a_raw(P, B),
               lambda P, k: F.fusedmm_a_backward_raw(P, A[:k], B, G[:k], need=(True, False))[0],
               lambda P, k: F.fusedmm_a_backward_values_raw(P, A[:k], B, G[:k], want_dA=True)[1],
               lambda P, k: F.sddmm_raw(P, A[:k], B)):
        got, want = fn(P, m), fn(few, 64)
        assert torch.equal(got[:want.shape[0]], want)
