"""Which kernel the choice takes for products whose operands come from memory, not from the caches: experts' products that stream their weights (measured, us, dot_mfma_kernel
/ dot_mid_kernel; three sets of inputs in turn).  No launch, addresses are not used."""
import pytest

import paper_2105_04663_amd as g
from tests.pin import MFMA, MID, PAIR, last, pinned


def _taken(E, M, K, N, align=8, fill=None):
    mesh, dims = g.Mesh((1,), (0,)), g.DotDims((0,), (0,), (2,), (1,))
    shapes = ((E, M, K), (E, K, N), (E, M, N))
    sh = [g.Sharding(s, (-1, -1, -1)) for s in shapes]
    bufs = [g.ShardBuf((1 << 40) + (i << 36), g.BF16, -(-s[2] // align) * align) for i, s in enumerate(shapes)]
    with pinned(dry_run=True):
        g.local_dot(mesh, dims, bufs[0], sh[0], bufs[1], sh[1], bufs[2], sh[2], 0, fill, 1 << 45, g.dot_workspace_bytes(mesh, dims, *sh, -1, fill is not None))
        return last()[0]


@pytest.mark.parametrize("E,M,K,N,align", [(8, 363, 2176, 3840, 8),        # 47 / 71
                                           (4, 369, 1600, 8064, 8),        # 37 / 55
                                           (16, 339, 1344, 6144, 8),       # 94 / 126
                                           (8, 279, 3968, 6016, 8),        # 140 / 178
                                           (16, 289, 1600, 5760, 2)])      # 104 / 131
def test_streamed_weights(E, M, K, N, align):
    assert _taken(E, M, K, N, align) == MFMA


@pytest.mark.parametrize("E,M,K,N", [(1, 2048, 1024, 2048), (4, 384, 1344, 768), (1, 1024, 2048, 4096)])
def test_operands_that_the_caches_hold(E, M, K, N):
    assert _taken(E, M, K, N, 8) == MID


# Up to 128 rows every weight is drawn once whatever the tile (us, dot_mfma_kernel / dot_mid_kernel / dot_split_kernel's best)
@pytest.mark.parametrize("E,M,K,N,fill", [(4, 35, 3640, 7781, [18, 25, 30, 35]),           # 63 / 46 / 67
                                          (16, 36, 4057, 1491, [24, 29, 34] * 5 + [28])])  # 69 / 46 / 68
def test_streamed_weights_of_few_rows(E, M, K, N, fill):
    assert _taken(E, M, K, N, 8, fill) == MID


# Beyond them, where 256 x 256 tiles leave half of the compute units idle (us, dot_mfma_kernel / dot_mid_kernel / dot_pair_kernel)
@pytest.mark.parametrize("E,M,K,N,fill", [(16, 272, 3760, 1280, [140, 250] * 7 + [230, 272]),       # 97 / 85 / 93
                                          (4, 193, 3200, 6898, [100, 190, 150, 193])])              # 68 / 65 / 67
def test_streamed_weights_in_few_tiles(E, M, K, N, fill):
    assert _taken(E, M, K, N, 8, fill) == MID


# A K-major lhs: experts' weight gradients of E x M x (fill) x N (us, dot_mfma_kernel / dot_mid_kernel / dot_pair_kernel)
@pytest.mark.parametrize("C,M,N,filled", [(924, 3648, 1152, [915, 555, 505, 788, 636, 553, 827, 901]),         # 64 / 57 / 53
                                          (580, 1152, 7104, [556, 539, 578, 528]),                              # 53 / 44 / 47
                                          (689, 1728, 2896, [559, 377, 368, 633, 484, 431, 539, 464])])         # 63 / 60 / 53
def test_weight_gradients(C, M, N, filled):
    E = len(filled)
    mesh, dims = g.Mesh((1,), (0,)), g.DotDims((0,), (0,), (1,), (1,))
    sh = [g.Sharding(s, (-1, -1, -1)) for s in ((E, C, M), (E, C, N), (E, M, N))]
    bufs = [g.ShardBuf((1 << 40) + (i << 36), g.BF16) for i in range(3)]
    with pinned(dry_run=True):
        g.local_dot(mesh, dims, bufs[0], sh[0], bufs[1], sh[1], bufs[2], sh[2], 0, filled, 1 << 45, g.dot_workspace_bytes(mesh, dims, *sh, -1, True))
        assert last()[0] in (MID, PAIR)


def test_a_buffer_that_several_partitions_share_counts_once():
    """A 4 x 8 mesh, 768 x 768 of the output each: 6 MB of lhs and 13 MB of rhs in all, each shard used by 8 or 4 partitions (counted for each of them, 100 MB)."""
    mesh, dims = g.Mesh((4, 8), tuple(range(32))), g.DotDims((), (), (1,), (0,))
    sh = [g.Sharding((3072, 1024), (0, -1)), g.Sharding((1024, 6144), (-1, 1)), g.Sharding((3072, 6144), (0, 1))]
    kept = {}
    bufs = [[g.ShardBuf(kept.setdefault((t, g.shard_bounds(mesh, sh[t], p)[0]), (1 << 40) + (len(kept) << 30)), g.BF16) for p in range(32)] for t in range(3)]
    taken = []
    for share in (True, False):
        if not share:
            bufs = [[g.ShardBuf((1 << 50) + ((t * 32 + p) << 30), g.BF16) for p in range(32)] for t in range(3)]
        with pinned(dry_run=True):
            g.grouped_dot(mesh, dims, bufs[0], sh[0], bufs[1], sh[1], bufs[2], sh[2], None, 1 << 45, g.dot_workspace_bytes(mesh, dims, *sh, -1, False))
            taken.append(last()[0])
    assert taken[0] != taken[1]
