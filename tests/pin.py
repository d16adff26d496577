"""Which contraction kernel the bf16 Dots of this thread take (csrc/testing.h): pinned for a test, or asked afterwards."""
import contextlib
import ctypes as C

import paper_2105_04663_amd as g

BY_RULE, SCALAR, MFMA, MID, SPLIT, PAIR = -1, 0, 1, 2, 3, 5


class _Launch(C.Structure):
    _fields_ = [("kernel", C.c_int32), ("row_blocks", C.c_int32), ("one_launch", C.c_int32), ("dry_run", C.c_int32),
                ("table_bytes", C.c_int64), ("sums_begin", C.c_int64), ("sums_end", C.c_int64),
                ("moved_back", C.c_int32), ("col_blocks", C.c_int32)]


def _pin(kernel, row_blocks, one_launch, dry_run=False, col_blocks=0):
    p = _Launch(kernel, row_blocks, one_launch, int(dry_run), col_blocks=col_blocks)
    assert g.load_library().gspmd_testing_pin(C.byref(p)) == 0


@contextlib.contextmanager
def pinned(kernel=BY_RULE, row_blocks=0, one_launch=BY_RULE, dry_run=False, col_blocks=0):
    """`dry_run`: Dots stop short of their launches; addresses are not used, so no GPU is needed."""
    _pin(kernel, row_blocks, one_launch, dry_run, col_blocks)
    try:
        yield
    finally:
        _pin(BY_RULE, 0, BY_RULE)


def _last():
    p = _Launch()
    assert g.load_library().gspmd_testing_last(C.byref(p)) == 0
    return p


def last():
    """(kernel, row blocks, one launch for a whole sum) of this thread's last Dot."""
    p = _last()
    return p.kernel, p.row_blocks, p.one_launch


def last_workspace():
    """(bytes of launch tables, begin and end of the partial sums or counters and slots) in the workspace of this thread's last Dot."""
    p = _last()
    return p.table_bytes, p.sums_begin, p.sums_end


def last_moved_back():
    """How many problems (members of a sum one by one) of this thread's last launch have their last tile column moved back."""
    return _last().moved_back


def last_col_blocks():
    """dot_split_kernel's column blocks in this thread's last Dot (others 0)."""
    return _last().col_blocks
