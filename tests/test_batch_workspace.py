"""Workspace sizes of batches stay within those a caller may have on record (a
buffer sized once, the fixed array of cqc_reconstruct_fd_noalloc): the sizes of
three batches in every precision, as they were when the tables of a batch had
one group per tile shape.  Host only."""
import ctypes
import os

import pytest

from paper_2012_02333_amd import _lib

pytestmark = pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="libcqc.so not built")
I32 = ctypes.c_int32

PAIRS = [([a, b], [k]) for a, b in [(3, 4), (4, 6), (4, 10), (5, 9), (7, 10), (8, 7), (9, 6), (6, 6), (10, 10)]
         for k in (1, 2, 3, 4)]
CHAINS = [([5, 4, 6], [1, 2]), ([6, 6, 6], [2, 2]), ([8, 8, 8], [3, 3]), ([4, 4, 4, 4], [1, 1, 1])] * 5


def _size(spec, prec):
    keep, arr = [], (_lib.CqcInstance * len(spec))()
    for i, (f, cuts) in enumerate(spec):
        up = [c for c, k in enumerate(cuts) for _ in range(k)]
        a = [(I32 * len(f))(*f), (I32 * len(up))(*up), (I32 * len(up))(*[u + 1 for u in up]), (I32 * sum(f))(*range(sum(f)))]
        ents = (ctypes.c_void_p * len(f))(*([4096] * len(f)))
        keep += a + [ents]
        arr[i] = _lib.CqcInstance(_lib.CqcCut(sum(f), len(f), len(up), *a), ents, 8192, None)
    nb = ctypes.c_size_t(0)
    dt = _lib.F64 if prec == "fp64" else _lib.F32
    assert _lib.lib().cqc_fd_workspace_size(arr, len(spec), dt, dt, _lib.PREC[prec], ctypes.byref(nb)) == 0
    return nb.value


@pytest.mark.parametrize("prec,pairs,chains,both", [
    ("fp64", 230656, 173454592, 173683968), ("fp32", 268032, 88353024, 88619520),
    ("bf16x6", 11740928, 246622464, 258361600), ("bf16x3", 7916288, 193865984, 201780480)])
def test_batch_workspace_no_larger(prec, pairs, chains, both):
    assert _size(PAIRS, prec) <= pairs
    assert _size(CHAINS, prec) <= chains
    assert _size(PAIRS + CHAINS, prec) <= both
