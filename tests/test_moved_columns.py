"""Members of a sum meet by tile and lane, not by column: the last tile column is moved back for all of them or for none, whatever the
row strides and base addresses of each (host only: Dots stop short of their launches)."""
import pytest

import paper_2105_04663_amd as g
from tests.pin import BY_RULE, MFMA, MID, last, last_moved_back, pinned


def _moved(M, K, N, strides, offsets, out_map, kernel, one_launch):
    P = len(strides)
    mesh, dims = g.Mesh((P,), tuple(range(P))), g.DotDims((), (), (1,), (0,))
    l, r, o = g.Sharding((M, K), (-1, 0)), g.Sharding((K, N), (0, -1)), g.Sharding((M, N), out_map)
    n = g.dot_workspace_bytes(mesh, dims, l, r, o)
    lhs = [g.ShardBuf((1 << 40) + (p << 36), g.BF16, 0) for p in range(P)]
    rhs = [g.ShardBuf((1 << 50) + (p << 36) + off, g.BF16, ld) for p, (ld, off) in enumerate(zip(strides, offsets))]
    out = [g.ShardBuf((1 << 55) + ((p << 36) if out_map == (-1, 0) else 0), g.BF16, 0) for p in range(P)]
    with pinned(kernel, 0, one_launch, dry_run=True):
        g.grouped_dot(mesh, dims, lhs, l, rhs, r, out, o, None, 1 << 30, n + (1 << 20))
    return last_moved_back()


@pytest.mark.parametrize("kernel", [MFMA, MID])
@pytest.mark.parametrize("strides,offsets", [((2056, 2050), (0, 0)), ((2050, 2056), (0, 0)), ((2056, 2056), (0, 4)), ((2056, 2056), (8, 0)),
                                             ((2056, 2056, 2058), (0, 0, 0)), ((2056, 2056), (0, 0)), ((2050, 2050), (0, 0))])
def test_all_members_or_none(strides, offsets, kernel):
    P = len(strides)
    loose = any(s % 8 for s in strides) or any(o % 16 for o in offsets)
    assert _moved(300, 512 * P, 2050, strides, offsets, (-1, -1), kernel, 1) == (P if loose else 0)
    assert last() == (kernel, 0, 1)
    # by themselves, each product by its own rows
    assert _moved(300, 512 * P, 2050, strides, offsets, (-1, -1), kernel, 0) == sum(1 for s, o in zip(strides, offsets) if s % 8 or o % 16)
    assert last() == (kernel, 0, 0)


@pytest.mark.parametrize("kernel", [MFMA, MID])
def test_pieces_of_a_scattered_sum(kernel):
    # owner 0's columns start at a multiple of 16 bytes, owner 1's 2050 elements further: with padded rows only the latter's pieces move
    assert _moved(300, 1024, 4100, (4104, 4104), (0, 0), (-1, 0), kernel, 1) == 2
    assert _moved(300, 1024, 4100, (4104, 4100), (0, 0), (-1, 0), kernel, 1) == 4
    assert last() == (kernel, 0, 1)


@pytest.mark.parametrize("M,K,N,strides,offsets", [(2048, 8192, 2050, (2056, 2050), (0, 0)), (4096, 4096, 4098, (4104, 4098), (0, 0)),
                                                   (2048, 8192, 2056, (2056, 2056), (0, 4))])
def test_by_rule(M, K, N, strides, offsets):
    assert _moved(M, K, N, strides, offsets, (-1, -1), BY_RULE, BY_RULE) == 2
