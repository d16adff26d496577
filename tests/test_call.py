"""The binding's native entry (csrc/call.c) takes Dots whose arguments are in their plain form and hands everything else back; either way a call
sees the present values, and comes to the same status as through ctypes (host only: launches are left out)."""
import sys
import threading

import numpy as np
import pytest

import paper_2105_04663_amd as g
from paper_2105_04663_amd import binding
from tests.pin import pinned


class _Recorder:
    """Stands in for the native entry and keeps what it returned."""

    def __init__(self, call):
        self.call, self.seen = call, []

    def __getattr__(self, name):
        def f(*a):
            self.seen.append(getattr(self.call, name)(*a))
            return self.seen[-1]
        return f


@pytest.fixture
def native(monkeypatch):
    g.load_library()
    assert binding._CALL is not None, "build the library first"
    rec = _Recorder(binding._CALL)
    monkeypatch.setattr(binding, "_CALL", rec)
    with pinned(dry_run=True):
        yield rec.seen


def _dot(P=4, fill=None):
    if fill:
        mesh, dims = g.Mesh((P,), tuple(range(P))), g.DotDims((0,), (0,), (2,), (1,))
        sh = [g.Sharding(s, (0, -1, -1)) for s in ((P, 64, 32), (P, 32, 48), (P, 64, 48))]
    else:
        mesh, dims = g.Mesh((P,), tuple(range(P))), g.DotDims((), (), (1,), (0,))
        sh = [g.Sharding((64, 32), (-1, -1)), g.Sharding((32, 200), (-1, 0)), g.Sharding((64, 200), (-1, 0))]
    bufs = [[g.ShardBuf((1 << 40) + (t * P + p << 30), g.BF16, 0) for p in range(P)] for t in range(3)]
    return mesh, dims, bufs, sh


def _run(mesh, dims, bufs, sh, fill=None, local=False, workspace=1 << 30, **more):
    n = g.dot_workspace_bytes(mesh, dims, *sh, -1, fill is not None)
    if local:
        g.local_dot(mesh, dims, bufs[0][0], sh[0], bufs[1][0], sh[1], bufs[2][0], sh[2], 0, fill, workspace, n, **more)
    else:
        g.grouped_dot(mesh, dims, bufs[0], sh[0], bufs[1], sh[1], bufs[2], sh[2], fill, workspace, n, **more)


@pytest.mark.parametrize("local", [False, True])
@pytest.mark.parametrize("P", [1, 4, 17, 40])
@pytest.mark.parametrize("fill", [False, True])
def test_plain_arguments_are_taken(native, P, fill, local):
    d = _dot(P, fill)
    _run(*d, fill=[7] * P if fill else None, local=local)
    _run(*d, fill=tuple([64] * P) if fill else None, local=local, epilogue=g.EPILOGUE_RELU, stream=0)
    assert native == [0, 0]


def test_what_is_not_plain_is_handed_back(native):
    mesh, dims, bufs, sh = _dot()

    class Buf(g.ShardBuf):
        pass

    changed = [
        ((g.Mesh([4], [0, 1, 2, 3]), dims, bufs, sh), {}),                                   # lists: may change in place
        ((g.Mesh((np.int64(4),), (0, 1, 2, 3)), dims, bufs, sh), {}),
        ((mesh, dims, bufs, [sh[0], sh[1], g.Sharding((64, np.int32(200)), (-1, 0))]), {}),
        ((mesh, dims, [[Buf(b.data, b.dtype) for b in bufs[0]], bufs[1], bufs[2]], sh), {}),
        ((mesh, dims, [[g.ShardBuf(b.data, np.int32(g.BF16)) for b in bufs[0]], bufs[1], bufs[2]], sh), {}),
        ((mesh, dims, [[g.ShardBuf(b.data, True) for b in bufs[0]], bufs[1], bufs[2]], sh), {}),
        ((mesh, dims, bufs, sh), {"epilogue": True}),
        ((mesh, dims, bufs, sh), {"epilogue": np.int64(1)}),
        ((mesh, dims, bufs, sh), {"stream": None}),
        ((mesh, dims, bufs, sh), {"workspace": np.int64(1 << 30)}),
    ]
    for args, more in changed:
        native.clear()
        try:
            _run(*args, **more)
        except (TypeError, g.GspmdError):
            pass                                     # what ctypes says to it
        assert native == [None], (args, more)
    native.clear()
    with pytest.raises(ValueError):
        _run(mesh, dims, [bufs[0][:3], bufs[1], bufs[2]], sh)
    with pytest.raises(TypeError):
        _run(mesh, dims, [[g.ShardBuf(4096.0, g.BF16)] * 4, bufs[1], bufs[2]], sh)
    assert native == [None, None]


@pytest.mark.parametrize("held", [False, True])
@pytest.mark.parametrize("P", [1, 4, 70])
def test_fewer_fill_counts_than_batch_entries(native, P, held):
    """One count is read for every batch entry, of one partition up to its last: a list that ends earlier would be read beyond its end."""
    mesh, dims, bufs, sh = d = _dot(P, fill=True)
    if held:
        _run(*d, fill=[64] * P)
        native.clear()
    for short in ([64] * (P - 1), (64,) * (P - 1), []):
        for call in (lambda: _run(*d, fill=short),
                     lambda: g.grouped_dot_noalloc(mesh, dims, bufs[0], sh[0], bufs[1], sh[1], bufs[2], sh[2], short),
                     lambda: g.resharded_dot(mesh, dims, bufs[0], sh[0], bufs[1], sh[1], bufs[2], sh[2], short, 1 << 30, 1 << 30),
                     lambda: g.local_dot(mesh, dims, bufs[0][0], sh[0], bufs[1][0], sh[1], bufs[2][0], sh[2], P - 1, short, 1 << 30, 4096),
                     lambda: g.plan_dot(mesh, dims, *sh, P - 1, lhs_fill=short)):
            with pytest.raises(ValueError):
                call()
    assert all(status is None for status in native)
    native.clear()
    _run(*d, fill=[64] * (P + 3))                    # more than are read
    _run(*d, fill=[64], local=True)                  # partition 0 reads the first alone
    assert len(g.plan_dot(mesh, dims, *sh, 0, lhs_fill=[64])) == 1
    assert native == [0, 0 if P == 1 else None]


def test_fill_counts_of_what_is_refused_anyway(native):
    mesh, dims, bufs, sh = _dot(4, fill=True)
    for m, d, s in ((g.Mesh((4,), (0, 1, 2, 2)), dims, sh), (mesh, g.DotDims((7,), (0,), (2,), (1,)), sh), (mesh, dims, [g.Sharding((4, 64, 32), (0, 0, -1))] + sh[1:])):
        with pytest.raises(g.GspmdError):
            g.local_dot(m, d, bufs[0][0], s[0], bufs[1][0], s[1], bufs[2][0], s[2], 0, [64], 1 << 30, 4096)


@pytest.mark.parametrize("local", [False, True])
def test_statuses_are_those_of_ctypes(native, local, monkeypatch):
    mesh, dims, bufs, sh = _dot()
    wrong = [
        ((mesh, dims, [[g.ShardBuf(b.data, g.F32) for b in bufs[0]], bufs[1], bufs[2]], sh), {}),                 # another type than the rhs's
        ((mesh, dims, bufs, sh), {"epilogue": 9}),
        ((mesh, dims, bufs, sh), {"workspace": 0}),
        ((mesh, dims, bufs, sh), {"workspace": (1 << 30) + 8}),
        ((mesh, dims, [[g.ShardBuf(b.data, g.BF16, 3) for b in bufs[0]], bufs[1], bufs[2]], sh), {}),
        ((mesh, dims, [[g.ShardBuf(0, g.BF16) for b in bufs[0]], bufs[1], bufs[2]], sh), {}),
        ((g.Mesh((4,), (0, 1, 2, 2)), dims, bufs, sh), {}),
        ((mesh, g.DotDims((), (), (0,), (0,)), bufs, sh), {}),
    ]
    def status(args, more):
        mesh, dims, (l, r, o), sh = args
        with pytest.raises(g.GspmdError) as e:
            if local:
                g.local_dot(mesh, dims, l[0], sh[0], r[0], sh[1], o[0], sh[2], 0, None, workspace_bytes=4096, **{"workspace": 1 << 30, **more})
            else:
                g.grouped_dot(mesh, dims, l, sh[0], r, sh[1], o, sh[2], None, workspace_bytes=4096, **{"workspace": 1 << 30, **more})
        return e.value.status, str(e.value)

    for args, more in wrong:
        status(args, more)                           # (the second time the descriptors' C form is held)
        plain = status(args, more)
        assert native[-1] == plain[0] != 0
        with monkeypatch.context() as m:
            m.setattr(binding, "_CALL", None)
            assert status(args, more) == plain


def test_present_values_count(native):
    mesh, dims, bufs, sh = _dot()
    _run(mesh, dims, bufs, sh)
    mesh.device_ids = (0, 1, 2, 2)                   # no permutation any more
    with pytest.raises(g.GspmdError):
        _run(mesh, dims, bufs, sh)
    mesh.device_ids = (3, 2, 1, 0)
    _run(mesh, dims, bufs, sh)
    bufs[1][2].dtype = g.F32
    with pytest.raises(g.GspmdError):
        _run(mesh, dims, bufs, sh)


def test_references_are_given_back(native):
    mesh, dims, bufs, sh = _dot(40, fill=True)
    fill = [1000 + i for i in range(40)]
    fill = [min(f, 64) for f in fill]
    _run(mesh, dims, bufs, sh, fill)
    watched = [mesh, dims, *sh, mesh.__dict__["_held"], sh[0].__dict__["_held"], bufs[0][0], bufs[0], fill]
    before = [sys.getrefcount(w) for w in watched]
    for _ in range(50):
        _run(mesh, dims, bufs, sh, fill)
        with pytest.raises(g.GspmdError):
            _run(mesh, dims, bufs, sh, fill, epilogue=9)
        _run(mesh, dims, bufs, sh, fill, local=True)
        try:
            _run(mesh, dims, bufs, sh, [1.5] * 40)
        except (TypeError, ValueError, g.GspmdError):
            pass
    assert [sys.getrefcount(w) for w in watched] == before


def test_fields_that_change_while_calls_run():
    g.load_library()
    mesh, dims, bufs, sh = _dot()
    stop, errors = threading.Event(), []

    def change():
        while not stop.is_set():
            mesh.device_ids = tuple([3, 2, 1, 0])
            mesh.device_ids = tuple([0, 1, 2, 3])

    def call():
        try:
            with pinned(dry_run=True):
                for _ in range(300):
                    _run(mesh, dims, bufs, sh)
        except Exception as e:                       # noqa: BLE001 - reported below
            errors.append(e)

    threads = [threading.Thread(target=call) for _ in range(3)]
    changer = threading.Thread(target=change)
    changer.start()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    stop.set()
    changer.join()
    assert not errors
