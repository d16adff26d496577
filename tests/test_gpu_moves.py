"""The shard copies and the resharding at the sizes where their 16-byte chunks can go wrong: rows that start at any
element of a 16-byte block, rows shorter than a chunk, chunks cut by a src shard's edge or by the valid extent, rows
that share a wave, one-dimensional and rank-4 tensors.  Values only move, so every comparison is bit for bit, against
slices of the global tensor at the oracle's bounds."""
import numpy as np
import pytest
import torch

import paper_2105_04663_amd as g
from oracle import bounds as ob

pytestmark = pytest.mark.gpu

CASES = [   # shape, mesh, src mapping, dst mapping
    ((7,), (3,), (0,), (-1,)), ((5000,), (4,), (-1,), (0,)), ((64, 8), (2,), (0, -1), (-1, 0)), ((33, 3), (2, 2), (0, 1), (1, 0)),
    ((13, 1031), (2, 3), (0, 1), (1, -1)), ((6, 5, 77), (2, 3), (0, -1, 1), (-1, 1, 0)), ((3, 4, 5, 130), (4, 2), (-1, 0, -1, 1), (1, -1, -1, 0)),
    ((130, 4099), (4, 8), (0, 1), (1, 0)), ((1, 9000), (5,), (-1, 0), (-1, -1)),
]


def buffers(mesh, sh, dtype, pitch, shift, fill):
    """Per partition: (handle, view of the static shard), the data starting `shift` elements into its allocation."""
    out = []
    for pid in range(mesh.n_partitions):
        _, _, shard = g.shard_bounds(mesh, sh, pid)
        last = shard[-1]
        ld = last + pitch if len(shard) > 1 else last
        rows = int(np.prod(shard[:-1], dtype=np.int64)) if len(shard) > 1 else 1
        t = torch.full((rows * ld + shift + 8,), fill, dtype=dtype, device="cuda")
        buf = g.ShardBuf(t.data_ptr() + shift * t.element_size(), g.BF16 if dtype == torch.bfloat16 else g.F32, ld if len(shard) > 1 else 0)
        out.append((buf, t, shard, ld, rows, shift))
    return out


def read(entry):
    _, t, shard, ld, rows, shift = entry
    return t[shift:shift + rows * ld].view(rows, ld)[:, :shard[-1]].reshape(shard).float().cpu().numpy()


def untouched(entry, fill):
    """Elements around the static shard: before it, after it, and between its rows."""
    _, t, shard, ld, rows, shift = entry
    gap = t[shift:shift + rows * ld].view(rows, ld)[:, shard[-1]:]
    return bool((torch.cat([t[:shift], t[shift + rows * ld:], gap.reshape(-1)]) == fill).all())


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("pitch,shift", [(0, 0), (0, 3), (5, 1), (3, 0)])
@pytest.mark.parametrize("shape,mesh_shape,smap,dmap", CASES)
def test_moves_at_any_alignment(shape, mesh_shape, smap, dmap, pitch, shift, dtype):
    P = int(np.prod(mesh_shape))
    ids = np.random.default_rng(P).permutation(P).tolist()
    mesh = g.Mesh(mesh_shape, tuple(ids))
    src_sh, dst_sh = g.Sharding(shape, smap), g.Sharding(shape, dmap)
    whole = torch.arange(int(np.prod(shape)), device="cuda").remainder(251).add(1).to(dtype).reshape(shape)
    ref = whole.float().cpu().numpy()
    stream = torch.cuda.current_stream().cuda_stream
    pad = -7.0
    bits = 0xC0E0 if dtype == torch.bfloat16 else 0xC0E00000      # -7
    src, dst = buffers(mesh, src_sh, dtype, pitch, shift, -3.0), buffers(mesh, dst_sh, dtype, (pitch * 3) % 7, (shift + 2) % 5, -3.0)

    def want(sh, pid, fill):
        off, valid, shard = ob.shard_bounds(mesh_shape, ids, shape, sh.dims_mapping, pid)
        w = np.full(shard, fill, dtype=np.float32)
        if all(valid):
            w[tuple(slice(0, n) for n in valid)] = ref[tuple(slice(o, o + n) for o, n in zip(off, valid))]
        return w

    for pid in range(P):
        g.shard_extract(mesh, src_sh, pid, whole.data_ptr(), src[pid][0], bits, stream)
        assert np.array_equal(read(src[pid]), want(src_sh, pid, pad)), f"extract {pid}"
        assert untouched(src[pid], -3.0), f"extract {pid}"
    n = g.reshard_workspace_bytes(mesh)
    ws = torch.empty(n + 256, dtype=torch.uint8, device="cuda")
    g.reshard(mesh, src_sh, [x[0] for x in src], dst_sh, [x[0] for x in dst], (ws.data_ptr() + 255) // 256 * 256, n, stream)
    back = torch.full((int(np.prod(shape)) + 16,), -3.0, dtype=dtype, device="cuda")
    at = 5                                                        # the global tensor starts anywhere too
    for pid in range(P):
        assert np.array_equal(read(dst[pid]), want(dst_sh, pid, 0.0)), f"reshard {pid}"
        assert untouched(dst[pid], -3.0), f"reshard {pid}"
        g.shard_assemble(mesh, dst_sh, pid, dst[pid][0], back.data_ptr() + at * back.element_size(), stream)
    flat = back.float().cpu().numpy()
    assert np.array_equal(flat[at:at + ref.size].reshape(shape), ref)
    assert (flat[:at] == -3.0).all() and (flat[at + ref.size:] == -3.0).all()


def test_extents_beyond_the_31_bit_kernel():
    # more than 2^30 elements in one dimension: element by element in 64-bit indices; shards start at odd elements
    n, P = (1 << 30) + 5, 3
    mesh, sh = g.Mesh((P,), (2, 0, 1)), g.Sharding((n,), (0,))
    whole = torch.empty(n, dtype=torch.int16, device="cuda").random_()
    back = torch.zeros_like(whole)
    stream = torch.cuda.current_stream().cuda_stream
    for pid in range(P):
        (off,), (valid,), (per,) = g.shard_bounds(mesh, sh, pid)
        t = torch.zeros(per + 2, dtype=torch.int16, device="cuda")
        buf = g.ShardBuf(t.data_ptr() + 2, g.BF16, 0)
        g.shard_extract(mesh, sh, pid, whole.data_ptr(), buf, 0x7FC0, stream)
        assert torch.equal(t[1:1 + valid], whole[off:off + valid]), f"extract {pid}"
        assert bool((t[1 + valid:1 + per] == 0x7FC0).all()) and int(t[0]) == 0 and int(t[-1]) == 0, f"extract {pid}"
        g.shard_assemble(mesh, sh, pid, buf, back.data_ptr(), stream)
    assert torch.equal(back, whole)
