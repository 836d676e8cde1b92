"""Attention vectors and features that are no contiguous arrays: columns of one matrix, and
every second row."""
import pytest
import torch

import paper_2203_07673_amd as F
from tests.gpu_helpers import log
from workloads import rmat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_strided_vectors(dtype):
    log(f"strided attention vectors {dtype}")
    S = rmat(8, 8, seed=931)
    P = F.Pattern.from_csr(S)
    gen = torch.Generator(device="cuda").manual_seed(932)
    H = torch.randn(S.n, 32, generator=gen, device="cuda").to(dtype)
    W = torch.randn(32, 2, generator=gen, device="cuda")
    G = torch.randn(S.m, 32, generator=gen, device="cuda")

    def head(a1, a2):
        a1, a2 = a1.detach().requires_grad_(True), a2.detach().requires_grad_(True)
        X = H.clone().requires_grad_(True)
        out = F.gat(P, X, a1, a2)
        return [out, *F.gat_scores(H, a1, a2), *torch.autograd.grad(out, (X, a1, a2), G)]

    want = head(W[:, 0].contiguous(), W[:, 1].contiguous())
    for a1, a2 in ((W[:, 0], W[:, 1]), (W[:, 0], W[:, 1].contiguous()), (W[:, 0].contiguous(), W[:, 1])):
        for x, y in zip(head(a1, a2), want):
            assert torch.equal(x, y)
    wide = torch.stack([H, torch.zeros_like(H)], 1).reshape(2 * S.n, 32)[::2]
    assert not wide.is_contiguous()
    for x, y in zip(F.gat_scores(wide, W[:, 0], W[:, 1]), want[1:3]):
        assert torch.equal(x, y)
