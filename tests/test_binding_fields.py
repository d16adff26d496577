"""The binding keeps the C form of meshes, shardings and dimension numbers between calls; whatever happens to the Python
objects in between, a call sees their present values (host only)."""
import copy
import pickle

import paper_2105_04663_amd as g


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
