"""Which contraction kernel the bf16 Dots of this thread take (csrc/testing.h): pinned for a test, or asked afterwards."""
import contextlib
import ctypes as C

import paper_2105_04663_amd as g

BY_RULE, SCALAR, MFMA, MID, SPLIT = -1, 0, 1, 2, 3


class _Launch(C.Structure):
    _fields_ = [("kernel", C.c_int32), ("row_blocks", C.c_int32), ("one_launch", C.c_int32)]


def _pin(kernel, row_blocks, one_launch):
    p = _Launch(kernel, row_blocks, one_launch)
    assert g.load_library().gspmd_testing_pin(C.byref(p)) == 0


@contextlib.contextmanager
def pinned(kernel=BY_RULE, row_blocks=0, one_launch=BY_RULE):
    _pin(kernel, row_blocks, one_launch)
    try:
        yield
    finally:
        _pin(BY_RULE, 0, BY_RULE)


def last():
    """(kernel, row blocks, one launch for a whole sum) of this thread's last Dot."""
    p = _Launch()
    assert g.load_library().gspmd_testing_last(C.byref(p)) == 0
    return p.kernel, p.row_blocks, p.one_launch
