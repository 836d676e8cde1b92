"""The attention head under saved-tensor hooks: what the forward keeps for the adjoint may come
back in another layout, and what comes back as something else is refused."""
import pytest
import torch

import paper_2203_07673_amd as F
from tests.gpu_helpers import log
from workloads import rmat

pytestmark = pytest.mark.gpu


def _head(softmax):
    S = rmat(8, 8, seed=921)
    gen = torch.Generator(device="cuda").manual_seed(922)
    H = torch.randn(S.n, 32, generator=gen, device="cuda", requires_grad=True)
    a1, a2 = (torch.randn(32, generator=gen, device="cuda").requires_grad_(True) for _ in range(2))
    P = F.Pattern.from_csr(S)
    G = torch.randn(S.m, 32, generator=gen, device="cuda")

    def run(pack, unpack):
        with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
            out = F.gat(P, H, a1, a2, softmax=softmax)
        return torch.autograd.grad(out, (H, a1, a2), G)

    return run


@pytest.mark.parametrize("softmax", [True, False])
def test_vectors_in_another_layout(softmax):
    log(f"saved scores softmax={softmax}")
    run = _head(softmax)
    want = run(lambda x: x, lambda x: x)

    def spread(x):  # every second element of a vector twice as long
        return x if x.dim() != 1 else torch.stack([x, torch.full_like(x, float("nan"))], 1).reshape(-1)[::2]

    for pack, unpack in ((spread, lambda x: x), (lambda x: x.detach().cpu(), lambda x: x.cuda())):
        for x, y in zip(run(pack, unpack), want):
            assert torch.equal(x, y)


def test_other_vectors_are_refused():
    log("saved scores refused")
    run = _head(True)
    with pytest.raises((TypeError, ValueError)):
        run(lambda x: x, lambda x: x.double() if x.dim() == 1 and x.numel() > 32 else x)
    with pytest.raises((TypeError, ValueError)):
        run(lambda x: x, lambda x: x[1:] if x.dim() == 1 and x.numel() > 32 else x)
