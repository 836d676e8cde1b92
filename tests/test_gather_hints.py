"""Gather hints reach the hardware: the kernels that follow them hold both loads of a gathered
row, with the streaming hint and without (the compiler can join the two into a plain one,
which no result shows), and their results have the bits of the kernels without hints."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest
import torch

import paper_2203_07673_amd as F
from paper_2203_07673_amd import _capi as C
from paper_2203_07673_amd import build
from tests.gpu_helpers import log

KERNELS = [  # operation, held / first / second gathered type, vectors a lane, elements a vector, entries a batch
    ("OP_FUSED1", "float", "float", "float", 1, 4, 4),
    ("OP_FUSED2", "float", "float", "float", 1, 4, 1),
    ("OP_FUSED1", "bf16_t", "bf16_t", "bf16_t", 1, 8, 4),
    ("OP_SPMM1", "float", "float", "float", 2, 4, 2),
]


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="needs hipcc")
def test_hinted_kernels_hold_both_loads(tmp_path):
    src = tmp_path / "hinted.hip"
    src.write_text('#include "fmm_lines.hpp"\n' + "".join(
        f"template __global__ void fmm::line_kernel<fmm::{op}, {h.replace('bf16', 'fmm::bf16')}, "
        f"{g1.replace('bf16', 'fmm::bf16')}, {g2.replace('bf16', 'fmm::bf16')}, float, 64, {nv}, {vw}, {u}, true>"
        "(fmm::LineArgs, int32_t);\n" for op, h, g1, g2, nv, vw, u in KERNELS))
    asm = tmp_path / "hinted.s"
    subprocess.run([build.HIPCC, *[f for f in build.FLAGS if f != "-fPIC"], "--cuda-device-only", "-S", "-o", str(asm),
                    str(src)], check=True, capture_output=True)
    bodies = re.split(r"^(_ZN3fmm11line_kernel\S+):", asm.read_text(), flags=re.M)[1:]
    assert len(bodies) == 2 * len(KERNELS)
    for (op, *_, nv, vw, u), name, body in zip(KERNELS, bodies[::2], bodies[1::2]):
        loads = re.findall(r"global_load_dwordx4 .*", body[:body.rindex("s_endpgm")])
        hinted = sum(1 for x in loads if re.search(r"\bnt\b", x))
        held = 0 if op == "OP_SPMM1" else nv  # loaded once, with the hint
        out = nv * vw // 4  # the output's old values (beta), plain
        assert hinted - held >= u * nv * (2 if op == "OP_FUSED2" else 1), (name, hinted, len(loads))
        assert hinted - held >= len(loads) - hinted - out, (name, hinted, len(loads))


@pytest.mark.gpu
@pytest.mark.parametrize("r,dtype", [(132, torch.float32), (256, torch.float32), (300, torch.float32),
                                     (1024, torch.float32), (264, torch.bfloat16), (1024, torch.bfloat16),
                                     (510, torch.float64)])
def test_hinted_rows_same_bits(r, dtype):
    """Every pass of 64 lanes a line, every batch depth, split and whole lines, with some, no
    and all entries hinted."""
    log(f"hinted rows r={r} {dtype}")
    rng = np.random.default_rng(3)
    m, n = 300, 200
    cols = [np.sort(rng.choice(n, size=k, replace=False)) for k in rng.integers(0, 40, m)]
    cols[7] = np.arange(n)
    ptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    acc = torch.float64 if dtype == torch.float64 else torch.float32
    val = torch.from_numpy(rng.random(ptr[-1])).to(acc)
    gen = torch.Generator(device="cuda").manual_seed(5)
    A, B = (torch.randn(k, r, generator=gen, device="cuda").to(dtype) for k in (m, n))
    G = torch.randn(m, r, generator=gen, device="cuda").to(acc)
    w = torch.rand(int(ptr[-1]), generator=gen, device="cuda").to(acc)

    def run(P):
        return [F.fusedmm_a_raw(P, A, B)[0], *F.fusedmm_a_backward_raw(P, A, B, G), F.sddmm_raw(P, A, B),
                F.spmm_a_raw(P, B, w), F.spmm_b_raw(P, A, w), *F.fusedmm_a_backward_values_raw(P, A, B, G, want_dA=True)]

    for variant in (1, 2, 3):
        P = F.Pattern(ptr, np.concatenate(cols).astype(np.int32), val, (m, n), val_dtype=acc, long_len=32, chunk=32)
        P.set_variant(variant, variant)
        assert P.launch_shape(C.FMM_CSR, False, r, F.dtype_code(A))[0] == 64
        want = run(P)
        for top in (20, 1, 400):
            for o in (C.FMM_CSR, C.FMM_CSC):
                P.set_gather_hints(o, top)
            for x, y in zip(run(P), want):
                assert torch.equal(x, y), (variant, top)
