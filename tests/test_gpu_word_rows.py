"""Operands whose rows are whole 32-bit words but not padded to 16 bytes (leading dimensions of an even number of elements that is no
multiple of 8): the direct variants of the 256 x 256 and the 128 x 128 tiles take them, a K-major rhs with its last tile column moved back.
Small integers and float32 output, compared bit for bit; everything beyond the valid extents holds NaN."""
import numpy as np
import pytest
import torch

import paper_2105_04663_amd as g
import workloads as wl
from oracle import dot as od
from tests.harness import Staged
from tests.pin import MFMA, MID, last, pinned

pytestmark = pytest.mark.gpu


def _workload(M, K, N, layout, Y):
    lhs_shape, rhs_shape = ((K, M) if layout & 1 else (M, K)), ((N, K) if layout & 2 else (K, N))
    return wl.DotWorkload(name="words", cfg=7, dtype="bf16", out_dtype="f32", lhs_shape=lhs_shape, rhs_shape=rhs_shape, lhs_batch=(), rhs_batch=(),
                          lhs_contract=(0,) if layout & 1 else (1,), rhs_contract=(1,) if layout & 2 else (0,), mesh_shape=(1, Y),
                          device_ids=tuple(range(Y)), lhs_map=(-1, -1), rhs_map=(1, -1) if layout & 2 else (-1, 1), out_map=(-1, 1))


@pytest.mark.parametrize("kernel", [MFMA, MID])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N,Y", [(256, 64, 256, 1), (300, 130, 257, 1), (40, 67, 511, 1), (520, 199, 770, 1), (130, 1000, 2 * 258 - 1, 2),
                                     (257, 321, 3 * 300 - 4, 3), (129, 33, 131, 1), (128, 31, 129, 1), (300, 70, 2 * 130, 2), (64, 701, 3 * 142 - 11, 3)])
def test_products(M, K, N, Y, layout, kernel):
    w = _workload(M, K, N, layout, Y)
    lhs, rhs = wl.draw_small_int_bf16(3, w.lhs_shape), wl.draw_small_int_bf16(4, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=2)
    with pinned(kernel):
        st.run_grouped()
        # dot_mid_kernel takes what is staged where a K-major lhs has a tile of rows
        if kernel == MFMA or not layout & 1 or M % 8 == 0 or M >= 128:
            assert last()[0] == kernel
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), (), (), w.lhs_contract, w.rhs_contract)
    for pid in range(Y):
        assert np.array_equal(st.out_shard(pid), od.expected_out_shard(ref, w.mesh_shape, w.device_ids, w.out_map, pid)), f"partition {pid}"


@pytest.mark.parametrize("kernel,one_launch", [(MFMA, 1), (MFMA, 0), (MID, 1), (MID, 0)])
@pytest.mark.parametrize("M,K,N,P", [(300, 402, 258, 2), (257, 1302, 770, 3), (130, 512, 334, 4)])
def test_sums_are_the_same_bits(M, K, N, P, kernel, one_launch):
    # N(0, 1) data: against the members' products with rows padded to 16 bytes, summed here in ascending order
    w = wl.ksplit(M=M, K=K, N=N, P=P)
    lhs, rhs = wl.draw_normal_bf16(5, w.lhs_shape), wl.draw_normal_bf16(6, w.rhs_shape)
    padded = Staged(w, lhs, rhs, row_align=8, out_dtype="f32")
    total = None
    for pid in range(P):
        tmp = torch.full((M * padded.out[pid][2],), float("nan"), device="cuda")
        padded.run_local(pid, out_override=g.ShardBuf.of(tmp, padded.out[pid][2]))
        part = tmp.view(M, -1)[:, :N].clone()
        total = part if total is None else total + part
    st = Staged(w, lhs, rhs, row_align=2, out_dtype="f32")
    with pinned(kernel, 0, one_launch):
        st.run_grouped()
        assert last() == (kernel, 0, one_launch)
    torch.cuda.synchronize()
    assert torch.equal(st.out[0][1].view(M, -1)[:, :N], total)


def _restride(st, pid, ld, first):
    """Partition `pid`'s rhs shard in rows of `ld` elements from element `first` of a buffer that ends with the last row's valid words."""
    _, old, old_ld, shard = st.rhs[pid]
    rows, cols = int(np.prod(shard[:-1])), shard[-1]
    t = torch.full((first + (rows - 1) * ld + (cols + 1) // 2 * 2,), float("nan"), dtype=torch.bfloat16, device="cuda")
    torch.as_strided(t, (rows, cols), (ld, 1), first).copy_(old.view(rows, old_ld)[:, :cols])
    st.keep.append(t)
    st.rhs[pid] = (g.ShardBuf.of(t[first:], ld), t, ld, shard)


@pytest.mark.parametrize("kernel,one_launch", [(MFMA, 1), (MFMA, 0), (MID, 1), (MID, 0)])
@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("strides,firsts", [((2056, 2052), (0, 0)), ((2052, 2056), (0, 0)), ((2056, 2056), (0, 2)), ((2056, 2056, 2058), (4, 0, 0)), ((2056, 2056), (0, 0))])
def test_members_with_rows_of_their_own(strides, firsts, scatter, kernel, one_launch):
    # one member's rhs rows are padded to 16 bytes, another's are not: all take the same columns for their last tile
    P, M, N = len(strides), 300, 2051             # scattered: 1026 and 1025 columns, 684, 684 and 683
    w = wl.ksplit(M=M, K=P * 256, N=N, P=P)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    w.out_map = (-1, 0) if scatter else (-1, -1)
    st = Staged(w, lhs, rhs, row_align=8, out_dtype="f32")
    for pid in range(P):
        _restride(st, pid, strides[pid], firsts[pid])
    room = torch.empty(1 << 26, dtype=torch.uint8, device="cuda")       # scattered pieces take more slots than the query has room for
    st.workspace = lambda *_: (room.data_ptr(), room.numel())
    with pinned(kernel, 0, one_launch):
        st.run_grouped()
        assert last() == (kernel, 0, one_launch)
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    for pid in range(P):
        assert np.array_equal(st.out_shard(pid), od.expected_out_shard(ref, w.mesh_shape, w.device_ids, w.out_map, pid)), f"partition {pid}"


@pytest.mark.parametrize("H", [300, 301, 512, 770])
@pytest.mark.parametrize("fill", [(10, 0, 257), (600, 17, 511)])
def test_rows_below_a_moved_tile_are_cleared(H, fill):
    # few occupied slots of 600; the output's rows are padded to 16 bytes, the rhs's are not
    w = wl.moe(E=3, C=600, M=64, H=H)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=8, out_dtype="bf16")
    _restride(st, 0, (H + 1) // 2 * 2, 0)
    with pinned(MFMA):
        st.run_grouped(fill=list(fill))
        assert last()[0] == MFMA
    got = st.out_shard(0)
    for e, f in enumerate(fill):
        want = wl.bf16_bits_to_f64(lhs)[e, :f] @ wl.bf16_bits_to_f64(rhs)[e]
        want = torch.from_numpy(want).to(torch.bfloat16).double().numpy()
        assert np.array_equal(got[e, :f], want) and not got[e, f:].any(), f"expert {e}"


def test_columns_right_of_a_moved_tile_are_cleared():
    # 770 columns over 3 partitions of 257: the last one has 256 valid of 257 static ones, with rows of 258
    w = _workload(300, 96, 770, 0, 3)
    lhs, rhs = wl.draw_normal_bf16(5, w.lhs_shape), wl.draw_normal_bf16(6, w.rhs_shape)
    for kernel in (MFMA, MID):
        st = Staged(w, lhs, rhs, row_align=2)
        for _, t, _, _ in st.out:
            t.fill_(float("nan"))
        with pinned(kernel):
            st.run_grouped()
        for pid in range(3):
            got = st.out_shard(pid)
            assert np.isfinite(got).all()
        assert (st.out_shard(2)[:, 256:] == 0).all()


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N,Y", [(128, 64, 129, 1), (131, 63, 257, 1), (300, 129, 3 * 141 - 1, 3), (129, 449, 2 * 131 - 1, 2), (257, 577, 131, 1), (133, 1345, 129, 1),
                                     (2101, 321, 2091, 1)])
def test_dense_odd_rows_through_registers(M, K, N, Y, layout):
    # every operand at odd element addresses: dot_mid_kernel's staged variant, at the edges of its tiles and of its ring of stages
    w = _workload(M, K, N, layout, Y)
    lhs, rhs = wl.draw_small_int_bf16(3, w.lhs_shape), wl.draw_small_int_bf16(4, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=0)
    with pinned(MID):
        st.run_grouped()
        assert last()[0] == MID
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), (), (), w.lhs_contract, w.rhs_contract)
    for pid in range(Y):
        assert np.array_equal(st.out_shard(pid), od.expected_out_shard(ref, w.mesh_shape, w.device_ids, w.out_map, pid)), f"partition {pid}"
