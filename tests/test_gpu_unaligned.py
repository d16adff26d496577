"""bf16 Dots on dense shards of any width, at any element address: the register-staged tiles fetch 16 bytes at element
alignment, move chunks that would reach past a row's end down in registers and take the last partial K tile element by
element.  Small integers and float32 output: every order of summation is exact, so results are compared bit for bit.
NaN lies right before and right after every operand."""
import numpy as np
import pytest
import torch

import paper_2105_04663_amd as g
import workloads as wl
from oracle import dot as od

pytestmark = pytest.mark.gpu

SIZES = [   # M, K, N: widths 1..7 past a multiple of 8, below 8, one to three tiles, K around 32- and 64-wide tiles
    (257, 33, 259), (300, 97, 261), (513, 64, 265), (270, 127, 515), (299, 160, 7), (5, 321, 300), (3, 1, 2), (258, 31, 263), (511, 1001, 254),
    (264, 200, 271), (300, 198, 262), (258, 130, 514), (100, 66, 1026),
]


def on_device(bits, rows, cols, shift):
    """A dense [rows, cols] array `shift` elements into an allocation that is NaN elsewhere."""
    t = torch.full((rows * cols + shift + 16,), float("nan"), dtype=torch.bfloat16, device="cuda")
    t[shift:shift + rows * cols] = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16).reshape(-1)
    return t, g.ShardBuf(t.data_ptr() + 2 * shift, g.BF16, 0)


@pytest.mark.parametrize("partial", [False, True])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("shift", [0, 1, 2])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_dense_rows_of_any_width(M, K, N, shift, layout, partial):
    # `partial`: the product as partition 0's partial sum of a contracting dimension of twice the size, which is never
    # left to the few-row kernel
    ls, rs = ((K, M) if layout & 1 else (M, K)), ((N, K) if layout & 2 else (K, N))
    lc, rc = ((0,) if layout & 1 else (1,)), ((1,) if layout & 2 else (0,))
    lhs, rhs = wl.draw_small_int_bf16(3, ls), wl.draw_small_int_bf16(4, rs)
    ta, a = on_device(lhs, *ls, shift)
    tb, b = on_device(rhs, *rs, (shift * 3) % 8)
    P = 2 if partial else 1
    mesh, dims = g.Mesh((P,), tuple(range(P))), g.DotDims((), (), lc, rc)
    def split(shape, dim):
        return g.Sharding(tuple(n * P if i == dim else n for i, n in enumerate(shape)), tuple(0 if i == dim and partial else -1 for i in (0, 1)))
    sh = [split(ls, lc[0]), split(rs, rc[0]), g.Sharding((M, N), (-1, -1))]
    n = g.dot_workspace_bytes(mesh, dims, *sh, 0)
    ws = torch.empty(n + 256, dtype=torch.uint8, device="cuda")
    out = torch.full((M * N + 8,), float("nan"), dtype=torch.float32, device="cuda")
    g.local_dot(mesh, dims, a, sh[0], b, sh[1], g.ShardBuf(out.data_ptr() + 4, g.F32, 0), sh[2], 0, None,
                (ws.data_ptr() + 255) // 256 * 256, n, torch.cuda.current_stream().cuda_stream)
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), (), (), lc, rc)
    got = out[1:1 + M * N].cpu().numpy().reshape(M, N)
    assert np.array_equal(got, ref)
    assert bool(torch.isnan(out[:1]).all()) and bool(torch.isnan(out[1 + M * N:]).all())


def test_partial_sums_of_odd_shards():
    # K split unevenly over 3 partitions, dense rows of 67 and 201: members share the output, so their sum is joined
    w = wl.ksplit(M=300, K=199, N=201, P=3)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    from tests.harness import Staged
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    for share in (True, False):
        st = Staged(w, lhs, rhs, row_align=0, out_dtype="f32", share_replicas=share)
        st.run_grouped()
        for pid in range(3):
            assert np.array_equal(st.out_shard(pid), ref)
