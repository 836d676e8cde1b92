"""Batch plans of both directions below and from 2^17 entries, where the forward and dA rows of a
tile begin to share a pass: the tiles, and the bits of single-graph calls."""
import numpy as np
import pytest
import torch

import paper_2203_07673_amd as F
from paper_2203_07673_amd import _capi as C
from tests.gpu_helpers import dev, log
from workloads import dense_normal

pytestmark = pytest.mark.gpu


def _pattern(m, n, entries, seed):
    rng = np.random.default_rng(seed)
    lens = np.full(m, entries // m)
    lens[:entries - lens.sum()] += 1
    first = rng.integers(0, n - lens.max(), m)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cols = (np.arange(entries) - np.repeat(rowptr[:-1], lens) + np.repeat(first, lens)).astype(np.int32)
    return F.Pattern(rowptr, cols, rng.random(entries).astype(np.float32), (m, n), split=False)


@pytest.mark.parametrize("r,dtype,dc", [(4, torch.float32, torch.float32), (72, torch.float32, torch.float32),
                                        (256, torch.float32, torch.float32), (8, torch.bfloat16, torch.float32),
                                        (96, torch.bfloat16, torch.bfloat16), (512, torch.bfloat16, torch.float32)])
@pytest.mark.parametrize("entries", [(1 << 17) - 1, 1 << 17])
def test_row_passes_by_size(r, dtype, dc, entries):
    log(f"batch by size r={r} {dtype} {dc} entries={entries}")
    sizes = [(4000, 3000, entries - 30000), (1500, 2500, 30000)]
    pats = [_pattern(m, n, e, 911 + k) for k, (m, n, e) in enumerate(sizes)]
    A = [dev(dense_normal(m, r, 912 + k)).to(dtype) for k, (m, _, _) in enumerate(sizes)]
    B = [dev(dense_normal(n, r, 914 + k)).to(dtype) for k, (_, n, _) in enumerate(sizes)]
    G = [dev(dense_normal(m, r, 916 + k)).to(dc) for k, (m, _, _) in enumerate(sizes)]
    both, fwd = F.BatchPlan(pats, A, B, G), F.BatchPlan(pats, A, B, forward=True, backward=False)
    bwd = F.BatchPlan(pats, A, B, G, forward=False)
    for placement in (both.PLACE_GLOBAL, both.PLACE_XCD, both.PLACE_QUEUES):
        for row_wave, col_wave in ((False, False), (True, False), (False, True), (True, True)):
            for p in (both, fwd, bwd):
                p.set_schedule(1536, placement, row_wave, col_wave)
                for x in (p.C or []) + (p.dA or []) + (p.dB or []):
                    x.fill_(float("nan"))
                p.run()
            n = [p.info()["n_tiles"] for p in (both, fwd, bwd)]
            assert n[0] == (n[1] + n[2] if entries < 1 << 17 else n[2]), n
            for x, y in zip(both.C + both.dA + both.dB, fwd.C + bwd.dA + bwd.dB):
                assert torch.equal(x, y)
    both.set_schedule(1536)
    both.run()
    for k, P in enumerate(pats):
        P.set_variant(C.FMM_VARIANT_DEEP, C.FMM_VARIANT_DEEP)
        c = F.fusedmm_a_raw(P, A[k], B[k])[0]
        dA, dB = F.fusedmm_a_backward_raw(P, A[k], B[k], G[k])
        assert torch.equal(both.C[k], c) and torch.equal(both.dA[k], dA) and torch.equal(both.dB[k], dB)


def test_workgroups_of_mixed_schedule():
    """Row-block rows with a wave per line in the column pass: no more than 5 workgroups a CU,
    for which the kernels are built."""
    P = _pattern(4000, 3000, 1 << 17, 911)
    r = 88
    plan = F.BatchPlan([P], [dev(dense_normal(4000, r, 1))], [dev(dense_normal(3000, r, 2))],
                       [dev(dense_normal(4000, r, 3))])
    for placement in (plan.PLACE_GLOBAL, plan.PLACE_XCD, plan.PLACE_QUEUES):
        plan.set_schedule(1536, placement, False, True)
        assert plan.info()["n_workgroups"] <= 5 * F.device_info()["num_cu"]
