"""The binding keeps the C form of meshes, shardings and dimension numbers between calls; whatever happens to the Python
objects in between, a call sees their present values (host only)."""
import copy
import ctypes as C
import pickle

import numpy as np
import pytest
import torch

import paper_2105_04663_amd as g
from paper_2105_04663_amd import binding


def test_present_values_count():
    mesh, sh = g.Mesh((2, 4), tuple(range(8))), g.Sharding((8, 64), (0, 1))
    first = g.shard_bounds(mesh, sh, 5)
    assert first == g.shard_bounds(mesh, sh, 5) == ((4, 16), (4, 16), (4, 16))
    mesh.device_ids = tuple(reversed(range(8)))                  # another tuple
    assert g.shard_bounds(mesh, sh, 5)[0] == (0, 32)
    sh.dims_mapping = (-1, 1)
    assert g.shard_bounds(mesh, sh, 5) == ((0, 32), (8, 16), (8, 16))
    ids = list(range(8))                                         # a list that changes in place
    mesh = g.Mesh((2, 4), ids)
    assert g.shard_bounds(mesh, sh, 5)[0] == (0, 16)
    ids.reverse()
    assert g.shard_bounds(mesh, sh, 5)[0] == (0, 32)


def test_copies_and_pickles():
    mesh, sh, dims = g.Mesh((4,), (0, 1, 2, 3)), g.Sharding((64, 90), (-1, 0)), g.DotDims((), (), (1,), (0,))
    g.dot_workspace_bytes(mesh, dims, g.Sharding((8, 64), (-1, -1)), sh, g.Sharding((8, 90), (-1, 0)))
    for m, s, d in ((copy.deepcopy(mesh), copy.copy(sh), copy.deepcopy(dims)), pickle.loads(pickle.dumps((mesh, sh, dims)))):
        assert (m, s, d) == (mesh, sh, dims)
        assert g.shard_bounds(m, s, 3) == g.shard_bounds(mesh, sh, 3)


@pytest.mark.parametrize("data", [torch.tensor(4096), np.int64(4096), 4096.0, "4096", C.c_void_p(4096)])
def test_only_an_address_is_an_address(data):
    # a tensor in place of its data_ptr() must not turn into an address by way of its value; one shard or several
    mesh, dims = g.Mesh((1,), (0,)), g.DotDims((), (), (1,), (0,))
    sh = g.Sharding((8, 8), (-1, -1))
    good, bad = g.ShardBuf(4096, g.BF16), g.ShardBuf(data, g.BF16)
    with pytest.raises(TypeError):
        g.grouped_dot(mesh, dims, [good], sh, [bad], sh, [good], sh)
    with pytest.raises(TypeError):
        g.local_dot(mesh, dims, good, sh, bad, sh, good, sh, 0)
    with pytest.raises(TypeError):
        g.reshard(mesh, sh, [good], sh, [bad])


@pytest.mark.parametrize("odd", [None, 2**63 + 5])        # an address beyond 63 bits takes another way
def test_shard_arrays_have_the_structures_layout(odd):
    bufs = [g.ShardBuf(odd, g.BF16, 8), g.ShardBuf(None, g.F32), g.ShardBuf(4096, np.int32(1), 2**40), g.ShardBuf(0, True, np.int64(3))]
    arr = (binding._CShardBuf * len(bufs)).from_buffer_copy(binding._bufs(bufs))
    for a, b in zip(arr, bufs):
        assert (a.data, a.dtype, a.row_stride) == (b.data or None, int(b.dtype), b.row_stride)


@pytest.mark.parametrize("dtype,row_stride", [(1.0, 0), (None, 0), (g.BF16, 8.0), (g.BF16, None), ("1", 0)])
def test_only_integers_describe_a_shard(dtype, row_stride):
    with pytest.raises(TypeError):
        binding._bufs([g.ShardBuf(4096, g.BF16), g.ShardBuf(4096, dtype, row_stride)])
