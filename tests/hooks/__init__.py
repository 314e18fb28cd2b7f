"""The scan's forms behind the rule that chooses between them (scan_forms.hip): two launches, or one with a given bound on the wait."""
import ctypes

from paper_2602_08686_amd import binding as B
from paper_2602_08686_amd import build

RULE = 1000   # units of 10 ns that the rule's form waits

_lib = None


def _load():
    global _lib
    if _lib is None:
        B.load()
        # they share structures: one built against an older library is not used
        if not build.HOOKS_LIB.exists() or build.HOOKS_LIB.stat().st_mtime < build.LIB.stat().st_mtime:
            build.build_test_hooks()
        lib, vp, n = ctypes.CDLL(str(build.HOOKS_LIB)), ctypes.c_void_p, ctypes.c_size_t
        pp = ctypes.POINTER(B.CkvParams)
        lib.hook_window_utility.argtypes = [pp] + [vp] * 8 + [n, ctypes.c_int, ctypes.c_uint32, vp]
        lib.hook_window_scores.argtypes = [pp] + [vp] * 4 + [n, ctypes.c_int, ctypes.c_uint32, vp]
        lib.hook_marks.argtypes = [pp, ctypes.POINTER(ctypes.c_int64)]
        lib.hook_marks.restype = ctypes.c_int64
        _lib = lib
    return _lib


def _at(*tensors):
    return [t.data_ptr() for t in tensors]


def window_utility(p, q, k, w_head, scratch, utility, budget, tau, ws, stream, two_launches=False, wait=RULE):
    st = _load().hook_window_utility(ctypes.byref(p), *_at(q, k, w_head, scratch, utility, budget, tau, ws), ws.numel(), two_launches,
                                     wait, stream.cuda_stream)
    assert st == B.CKV_OK, st


def window_scores(p, q, k, scores, ws, stream, two_launches=False, wait=RULE):
    st = _load().hook_window_scores(ctypes.byref(p), *_at(q, k, scores, ws), ws.numel(), two_launches, wait, stream.cuda_stream)
    assert st == B.CKV_OK, st


def marks(p):
    """(offset in the workspace, count) of a call's marks, eight bytes each; a count of 0 where the rule takes two launches."""
    offset = ctypes.c_int64(0)
    count = _load().hook_marks(ctypes.byref(p), ctypes.byref(offset))
    return offset.value, count
