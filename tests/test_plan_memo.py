"""Plans kept per thread: a call whose cut differs in any field gets its own
plan, pointers and workspace sizes are checked on every call, and more cuts
than the memo holds, in any order and from several threads, give the sizes a
fresh process gives."""
import ctypes
import itertools
import threading

import pytest

cqc = pytest.importorskip("paper_2012_02333_amd")
from paper_2012_02333_amd import _lib  # noqa: E402


def _size(cut, in_t=_lib.F32, prec=1, bwd=False):
    ptrs = (ctypes.c_void_p * cut.n_sub)()
    inst = (_lib.CqcInstance * 1)(_lib.CqcInstance(cut.c, ptrs, None, None))
    nb = ctypes.c_size_t(0)
    L = _lib.lib()
    rc = (L.cqc_backward_workspace_size(inst, 1, in_t, prec, ctypes.byref(nb)) if bwd else
          L.cqc_fd_workspace_size(inst, 1, in_t, in_t, prec, ctypes.byref(nb)))
    assert rc == 0
    return int(nb.value)


def _cuts():
    return [cqc.CutMap(9, [4, 5], [(0, 1)], list(range(9))), cqc.CutMap(9, [5, 4], [(0, 1)], list(range(9))),
            cqc.CutMap(9, [4, 5], [(0, 1)] * 2, list(range(9))), cqc.CutMap(9, [4, 5], [(1, 0)], list(range(9))),
            cqc.CutMap(9, [4, 5], [(0, 1)], [8, 7, 6, 5, 4, 3, 2, 1, 0]),
            cqc.CutMap(9, [3, 3, 3], [(0, 1), (1, 2)], list(range(9))),
            cqc.CutMap(9, [3, 3, 3], [(0, 1), (0, 2)], list(range(9)))]


@pytest.mark.parametrize("bwd", [False, True])
def test_sizes_do_not_depend_on_the_calls_before(bwd):
    variants = [(c, t, p) for c in _cuts() for t, p in ((_lib.F32, 1), (_lib.F64, 0), (_lib.F32, 0))]
    fresh = {}

    def one(i, c, t, p):   # a new thread starts with an empty memo
        fresh[i] = _size(c, t, p, bwd)

    for i, v in enumerate(variants):
        th = threading.Thread(target=one, args=(i, *v))
        th.start()
        th.join()
    for i, j in itertools.permutations(range(len(variants)), 2):
        assert _size(*variants[i], bwd) == fresh[i]
        assert _size(*variants[j], bwd) == fresh[j]


def test_kept_plan_still_checks_pointers_and_workspace():
    cut = _cuts()[0]
    need = _size(cut)
    L = _lib.lib()
    ptrs = (ctypes.c_void_p * 2)(0x1000, None)
    inst = (_lib.CqcInstance * 1)(_lib.CqcInstance(cut.c, ptrs, 0x1000, None))
    assert L.cqc_reconstruct_fd(inst, 1, _lib.F32, _lib.F32, 1, 0x1000, need, None) == 1
    ptrs[1] = 0x1000
    inst[0].out = None
    assert L.cqc_reconstruct_fd(inst, 1, _lib.F32, _lib.F32, 1, 0x1000, need, None) == 1
    inst[0].out = 0x1000
    assert L.cqc_reconstruct_fd(inst, 1, _lib.F32, _lib.F32, 1, 0x1000, need - 1, None) == 4
