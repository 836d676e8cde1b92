"""One pattern used from two streams or threads at a time: workspaces are kept by both, so the
partial sums of split lines, the attention adjoint's arrays and the solver's vectors of
overlapping calls do not meet."""
import threading

import pytest
import torch

import paper_2203_07673_amd as F
from paper_2203_07673_amd import _capi as C
from tests.gpu_helpers import log
from workloads import rmat

pytestmark = pytest.mark.gpu


def _workspaces(P, Q, out):
    out += [R.workspace(C.FMM_OP_FUSEDMM_A, 64, C.FMM_F32) for R in (P, Q)] + \
           [R._gat_workspace(True, 64, C.FMM_F32) for R in (P, Q)]


def test_workspaces_by_stream_and_thread():
    log("workspaces of their own")
    P = F.Pattern.from_csr(rmat(9, 8, seed=901), long_len=8, chunk=8)
    Q = P.with_values(P.val * 2)
    held = []  # two workspaces each, which the copy with other values shares
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            _workspaces(P, Q, held)
    t = threading.Thread(target=_workspaces, args=(P, Q, held))
    t.start()
    t.join()
    assert len(held) == 16 and all(ws.numel() == size > 0 for ws, size in held)
    assert len({ws.data_ptr() for ws, _ in held}) == 8
    kept = []
    _workspaces(P, Q, kept)
    assert [ws.data_ptr() for ws, _ in kept] == [ws.data_ptr() for ws, _ in held[:4]]
    # the solver's vectors and its partial sums are not one array, whatever their sizes
    assert P._scratch(4096, "cg").data_ptr() != P._scratch(4096).data_ptr()
    for k in range(3 * F.fusedmm.SCRATCH_KEPT):
        P._scratch(256 + k)
    assert len(P._ws_cache) <= F.fusedmm.SCRATCH_KEPT


def test_captured_calls_have_the_graphs_memory():
    """Eager calls between the replays of a captured one, on the stream of the capture."""
    log("captured workspaces")
    S = rmat(10, 12, seed=904)
    P = F.Pattern.from_csr(S, long_len=8, chunk=8)
    A, B, X = (torch.randn(S.m, 64, device="cuda", generator=torch.Generator("cuda").manual_seed(905 + k)) for k in range(3))
    out = torch.empty(S.m, 64, device="cuda")
    want, other = F.fusedmm_a_raw(P, A, B)[0], F.fusedmm_a_raw(P, X, B)[0]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        F.fusedmm_a_raw(P, A, B, out=out)
    torch.cuda.synchronize()
    kept = dict(P._ws_cache)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        F.fusedmm_a_raw(P, A, B, out=out)
    assert P._ws_cache.keys() == kept.keys()
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        with torch.cuda.stream(side):
            got = F.fusedmm_a_raw(P, X, B)[0]
        torch.cuda.synchronize()
        assert torch.equal(got, other)


@pytest.mark.parametrize("kind", ["fused", "attention", "als"])
def test_two_streams_at_a_time(kind):
    log(f"two streams {kind}")
    S = rmat(13, 16, seed=902)
    P = F.Pattern.from_csr(S, long_len=32, chunk=32)
    r = 64
    gen = torch.Generator(device="cuda").manual_seed(903)
    ins = [[torch.randn(S.m, r, generator=gen, device="cuda") for _ in range(3)] +
           [torch.randn(r, generator=gen, device="cuda") for _ in range(2)] for _ in range(2)]

    def call(x):
        A, B, G, a1, a2 = x
        if kind == "fused":
            return [F.fusedmm_a_raw(P, A, B)[0], *F.fusedmm_a_backward_raw(P, A, B, G), F.spmm_b_raw(P, A)]
        if kind == "attention":
            lse = torch.empty(S.m, device="cuda")
            out = F.gat_forward(P, A, a1, a2, lse=lse)
            return [out, *F.gat_backward(P, A, a1, a2, out, G, want_dS=True, lse=lse)]
        X, Y = G.clone(), B.clone()
        F.als_sweep(P, X, Y, 0.1, 3)
        return [X, Y, F.als_residual(P, X, Y)]

    want = [call(x) for x in ins]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in ins]
    got = [[], []]
    for _ in range(20):
        for k, st in enumerate(streams):
            with torch.cuda.stream(st):
                got[k].append(call(ins[k]))
    torch.cuda.synchronize()
    for k in range(2):
        for out in got[k]:
            for x, y in zip(out, want[k]):
                assert torch.equal(x, y), k
