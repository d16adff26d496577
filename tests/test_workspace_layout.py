"""What a grouped Dot lays out in its workspace -- launch tables, partial sums, counters and slots -- does not overlap and does not
leave the workspace (host only: Dots stop short of their launches)."""
import pytest

import paper_2105_04663_amd as g
from tests.pin import BY_RULE, MFMA, MID, last, last_workspace, pinned


def run(M, K, N, P, out_map, row_align, kernel, one_launch, extra):
    mesh, dims = g.Mesh((P,), tuple(range(P))), g.DotDims((), (), (1,), (0,))
    l, r, o = g.Sharding((M, K), (-1, 0)), g.Sharding((K, N), (0, -1)), g.Sharding((M, N), out_map)
    n = g.dot_workspace_bytes(mesh, dims, l, r, o)
    address = iter(range(1 << 40, 1 << 60, 1 << 36))

    def bufs(sh, one=False):
        last_dim = g.shard_bounds(mesh, sh, 0)[2][-1]
        ld = -(-last_dim // row_align) * row_align if row_align else 0
        out = [g.ShardBuf(next(address), g.BF16, ld) for _ in range(1 if one else P)]
        return out * P if one else out

    with pinned(kernel, 0, one_launch, dry_run=True):
        g.grouped_dot(mesh, dims, bufs(l), l, bufs(r), r, bufs(o, out_map == (-1, -1)), o, None, 1 << 30, n + extra)
    table, begin, end = last_workspace()
    assert table <= begin or begin == end, (last(), last_workspace())
    assert max(table, end) <= n + extra
    return last()


@pytest.mark.parametrize("kernel,one_launch", [(BY_RULE, BY_RULE), (MFMA, 1), (MFMA, 0), (MID, 1), (MID, 0)])
@pytest.mark.parametrize("out_map", [(-1, -1), (-1, 0)])
@pytest.mark.parametrize("P", [2, 4, 5, 6, 8, 16])
@pytest.mark.parametrize("extra", [0, 1 << 20])
def test_tables_and_sums_do_not_overlap(P, out_map, kernel, one_launch, extra):
    for M, K, N in ((742, 8448, 4032), (256, 4096, 256 * P), (2560, 512 * P, 256 * P), (300, 999, 2051), (64, 5, 40)):
        for row_align in (8, 0):
            run(M, K, N, P, out_map, row_align, kernel, one_launch, extra)


def test_sums_of_many_scattered_pieces_take_slots_where_there_is_room():
    assert run(256, 4096, 2048, 8, (-1, 0), 8, MFMA, 1, 1 << 20) == (MFMA, 0, 1)
    assert run(256, 4096, 2048, 8, (-1, 0), 8, MFMA, 1, 0)[2] == 0         # the query has no room for 64 pieces' table beside the slots
    assert run(256, 4096, 1024, 4, (-1, 0), 8, MFMA, 1, 0) == (MFMA, 0, 1)  # 16 pieces travel as kernel arguments
