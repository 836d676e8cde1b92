"""Attention rows whose softmax has no finite normaliser: split rows and whole rows agree."""
import numpy as np
import pytest
import torch

import paper_2203_07673_amd as F
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [1, 5, 16, 50, 64, 260])
@pytest.mark.parametrize("many", [False, True])
def test_split_rows_like_whole_ones(r, many):
    """A NaN edge value, all edges at minus infinity, one of them, one at plus infinity, and
    values at the type's lowest: NaN where the definition has no value, in split rows too."""
    log(f"softmax without a normaliser r={r} many={many}")
    k, deg = 6, 40
    m = 70000 if many else 200  # enough lines for merges by lane groups, or few
    rows = np.full(m, 0)
    rows[:k] = deg
    if many:
        rows[k:] = 6
    ptr = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    cols = np.concatenate([np.arange(d) for d in rows]).astype(np.int32)
    val = np.random.default_rng(941).random(ptr[-1]).astype(np.float32) + 0.5
    edge = [val[ptr[i]:ptr[i + 1]] for i in range(k)]
    edge[0][17] = np.nan
    edge[1][:] = -np.inf
    edge[2][3] = -np.inf
    edge[3][30] = np.inf
    edge[4][:] = np.finfo(np.float32).min
    gen = torch.Generator(device="cuda").manual_seed(942)
    H = torch.rand(m, r, generator=gen, device="cuda") + 0.5
    a = torch.full((r,), 1.0 / r, device="cuda")
    out = []
    for split in (False, True):
        P = F.Pattern(ptr, cols, val, (m, m), split=split, long_len=4, chunk=4)
        assert bool(P.schedules["csr"]) == split
        lse = torch.empty(m, device="cuda")
        out.append((F.gat_forward(P, H, a, a, lse=lse), lse))
    (whole, lw), (cut, lc) = out
    assert torch.isnan(whole[0]).all() and torch.isnan(whole[1]).all()
    assert torch.equal(torch.isnan(whole), torch.isnan(cut))
    fin = ~torch.isnan(whole)
    assert torch.isfinite(whole[fin]).all()
    assert torch.allclose(whole[fin], cut[fin], rtol=1e-5, atol=0)
    ok = torch.isfinite(whole).all(1)
    assert torch.allclose(lw[ok], lc[ok], rtol=1e-5, atol=1e-5)
