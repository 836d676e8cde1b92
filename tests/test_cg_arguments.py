"""The batched solves refuse a pattern or rows that their kernels could not read, before any
device work, like every other call."""
import ctypes

import pytest

from paper_2203_07673_amd import _capi as C
from tests.test_capi import FAKE, _desc

OK_SPLIT = dict(long_len=4, n_chunks=10, n_splits=2, chunks=FAKE, splits=FAKE)


def _solve(entry, d, F=FAKE, r=32, dtype=C.FMM_F32, ws=FAKE):
    lib = C.load()
    need = ctypes.c_size_t(0)
    assert lib.fmm_cg_work_size(d.rows, r, ctypes.byref(need)) == 0
    head = (ctypes.byref(d), F, r, dtype) + ((FAKE,) if entry == "fmm_cg_lines" else ())
    return getattr(lib, entry)(*head, 0.5, 3, FAKE, FAKE, need.value, ws, 1 << 20, None)


@pytest.mark.parametrize("entry", ["fmm_cg_lines", "fmm_als_lines"])
def test_unreadable_patterns(entry):
    for broken, status in ((dict(ptr=None), -1), (dict(idx=None), -1), (dict(nnz=-1), -2), (dict(n_chunks=-1), -2),
                           (dict(OK_SPLIT, chunks=None), -1), (dict(OK_SPLIT, splits=None), -1),
                           (dict(OK_SPLIT, long_len=0), -2), (dict(OK_SPLIT, n_splits=0), -2)):
        d = _desc()
        for k, v in broken.items():
            setattr(d, k, v)
        assert _solve(entry, d) == status, broken
    d = _desc()
    for k, v in OK_SPLIT.items():
        setattr(d, k, v)
    assert _solve(entry, d, ws=None) == -7
    # bfloat16 rows are read in 16-byte vectors
    assert _solve(entry, _desc(), F=FAKE + 2, dtype=C.FMM_BF16) == -8
    assert _solve(entry, _desc(), F=None) == -1
