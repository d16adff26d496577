"""dot_mid_kernel (128 x 128 tiles) at the edges of its tiles, of its LDS stages and of the 32-wide K tiles, in all four
operand layouts, and its sums over a contracting mesh dimension (members one after the other in one workgroup).  Every
product is given as a partial sum of a contracting dimension, so that the few-row kernel does not take it; small
integers and float32 output: compared bit for bit."""
import numpy as np
import pytest
import torch

import paper_2105_04663_amd as g
import workloads as wl
from oracle import dot as od
from tests import test_gpu_parity as parity
from tests.harness import Staged, out_tensor
from tests.pin import MFMA, MID, last, pinned

pytestmark = pytest.mark.gpu

SIZES = [   # M, K, N: K of 0 to 13 whole tiles with and without a partial one
    (128, 32, 128), (129, 31, 127), (1, 33, 300), (130, 64, 8), (200, 95, 136), (257, 128, 129), (127, 160, 384), (300, 161, 260), (140, 192, 64),
    (260, 200, 70), (64, 224, 500), (384, 416, 256), (100, 500, 100),
]


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_partial_product(M, K, N, layout):
    lhs_shape, rhs_shape = ((2 * K, M) if layout & 1 else (M, 2 * K)), ((N, 2 * K) if layout & 2 else (2 * K, N))
    lc, rc = ((0,) if layout & 1 else (1,)), ((1,) if layout & 2 else (0,))
    w = wl.DotWorkload(name="mid", cfg=7, dtype="bf16", out_dtype="f32", lhs_shape=lhs_shape, rhs_shape=rhs_shape, lhs_batch=(), rhs_batch=(),
                       lhs_contract=lc, rhs_contract=rc, mesh_shape=(2,), device_ids=(1, 0),
                       lhs_map=(0, -1) if layout & 1 else (-1, 0), rhs_map=(-1, 0) if layout & 2 else (0, -1), out_map=(-1, -1))
    lhs, rhs = wl.draw_small_int_bf16(3, lhs_shape), wl.draw_small_int_bf16(4, rhs_shape)
    st = Staged(w, lhs, rhs, row_align=8, share_replicas=False)       # row padding holds NaN
    a, b = wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs)
    dims = (w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    for pid in range(2):
        st.run_local(pid)
        assert np.array_equal(st.out_shard(pid), od.expected_partial(a, b, dims, w.mesh_shape, w.device_ids, w.lhs_map, w.rhs_map, pid))
        assert bool(torch.isnan(st.out[pid][1].view(M, -1)[:, N:]).all())


@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,N,P", [(300, 999, 264, 3), (129, 2048, 520, 8), (500, 70, 130, 4), (257, 33, 200, 5)])
def test_sums_of_members(M, K, N, P, out_dtype, scatter):
    # K split unevenly (with (257, 33, .., 5) the last member has 5 of 7 positions, with (500, 70, .., 4) 16 of 18)
    w = wl.ksplit(M=M, K=K, N=N, P=P)
    w.out_map = (-1, 0) if scatter else (-1, -1)
    lhs, rhs = wl.draw_normal_bf16(5, w.lhs_shape), wl.draw_normal_bf16(6, w.rhs_shape)
    whole = wl.ksplit(M=M, K=K, N=N, P=P)
    st = Staged(whole, lhs, rhs, row_align=8, out_dtype="f32", share_replicas=True)
    total = None
    for pid in range(P):                                              # ((p0 + p1) + p2) + .. of the members' own products
        tmp = torch.full((M * st.out[pid][2],), float("nan"), device="cuda")
        st.run_local(pid, out_override=g.ShardBuf.of(tmp, st.out[pid][2]))
        part = tmp.view(M, -1)[:, :N].clone()
        total = part if total is None else total + part
    total = total.clamp_min(0)
    st2 = Staged(w, lhs, rhs, row_align=8, out_dtype=out_dtype)
    st2.run_grouped(epilogue=1)
    torch.cuda.synchronize()
    per = -(-N // P)
    for pid in range(P):
        got = out_tensor(st2, pid)
        want = torch.zeros(got.shape, device="cuda")
        cols = total[:, pid * per:(pid + 1) * per] if scatter else total
        want[:, :cols.shape[1]] = cols
        assert torch.equal(got, want.to(got.dtype)), f"partition {pid}"


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", [(130, 448, 140), (100, 512, 300), (257, 576, 129), (129, 673, 264), (128, 1344, 130),      # one workgroup on a compute unit
                                   (2100, 320, 2090), (2100, 512, 2090), (2100, 735, 2090)])                                 # 289 tiles: two
def test_loads_around_the_ring_of_stages(M, K, N, layout):
    # K of as many 64-wide steps as the loop takes at a time, one more or less, with and without something left
    lhs_shape, rhs_shape = ((K, M) if layout & 1 else (M, K)), ((N, K) if layout & 2 else (K, N))
    lc, rc = ((0,) if layout & 1 else (1,)), ((1,) if layout & 2 else (0,))
    w = wl.DotWorkload(name="mid", cfg=7, dtype="bf16", out_dtype="f32", lhs_shape=lhs_shape, rhs_shape=rhs_shape, lhs_batch=(), rhs_batch=(),
                       lhs_contract=lc, rhs_contract=rc, mesh_shape=(1,), device_ids=(0,), lhs_map=(-1, -1), rhs_map=(-1, -1), out_map=(-1, -1))
    lhs, rhs = wl.draw_small_int_bf16(3, lhs_shape), wl.draw_small_int_bf16(4, rhs_shape)
    st = Staged(w, lhs, rhs, row_align=8)
    with pinned(MID):
        st.run_grouped()
        assert last()[0] == MID
    a, b = wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs)
    assert np.array_equal(st.out_shard(0), od.dot_general(a, b, (), (), lc, rc))


@pytest.mark.parametrize("M,N", [(130, 264), (2100, 2090)])
@pytest.mark.parametrize("per,P", [(64, 2), (64, 8), (128, 3), (192, 4), (320, 2), (704, 3), (96, 4), (33, 5), (70, 8), (254, 2), (639, 3)])
@pytest.mark.parametrize("short", [0, 1, 30])
def test_alike_members_follow_on(M, N, per, P, short):
    # members of equal K, the last one's equal or less: of 1 to 11 steps, the last one whole or not, the next ones' loads under way before the first is multiplied
    w = wl.ksplit(M=M, K=per * P - short, N=N, P=P)          # K beyond the last member's is padding
    lhs, rhs = wl.draw_normal_bf16(5, w.lhs_shape), wl.draw_normal_bf16(6, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=8, out_dtype="f32")
    got = {}
    for kernel, one in ((MID, 1), (MFMA, 0)):            # in one launch, and as dense partials of the 256 x 256 kernel and their sum
        st.out[0][1].fill_(float("nan"))
        with pinned(kernel, 0, one):
            st.run_grouped()
            assert last() == (kernel, 0, one)
        torch.cuda.synchronize()
        got[kernel] = st.out[0][1].view(M, -1)[:, :N].clone()
    assert torch.equal(got[MID], got[MFMA])
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    parity.check(st.out_shard(0), ref)


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,row_align", [(2100, 2090, 8), (2100, 2090, 2), (200, 300, 2)])       # two workgroups on a compute unit, one
@pytest.mark.parametrize("per", [33, 55, 64 + 40, 64 + 63, 128 + 31])
def test_what_is_left_of_members(M, N, row_align, per, layout):
    # one or two 32-wide tiles after each member's 64-wide steps, and no step before them
    K, P = 2 * per, 2
    lhs_shape, rhs_shape = ((K, M) if layout & 1 else (M, K)), ((N, K) if layout & 2 else (K, N))
    w = wl.DotWorkload(name="mid", cfg=7, dtype="bf16", out_dtype="f32", lhs_shape=lhs_shape, rhs_shape=rhs_shape, lhs_batch=(), rhs_batch=(),
                       lhs_contract=(0,) if layout & 1 else (1,), rhs_contract=(1,) if layout & 2 else (0,), mesh_shape=(P,), device_ids=(0, 1),
                       lhs_map=(0, -1) if layout & 1 else (-1, 0), rhs_map=(-1, 0) if layout & 2 else (0, -1), out_map=(-1, -1))
    lhs, rhs = wl.draw_small_int_bf16(5, lhs_shape), wl.draw_small_int_bf16(6, rhs_shape)
    st = Staged(w, lhs, rhs, row_align=row_align)
    with pinned(MID, 0, 1):
        st.run_grouped()
        if row_align == 8 or not layout & 1:          # (a K-major lhs takes 16-byte aligned rows only)
            assert last() == (MID, 0, 1)
    a, b = wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs)
    assert np.array_equal(st.out_shard(0), od.dot_general(a, b, (), (), w.lhs_contract, w.rhs_contract))


@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("N", [264, 301])
def test_sum_into_shards_of_different_strides(N, scatter, out_dtype):
    # a sum in two launches into every member's own out buffer, each with rows of its own
    M, K, P = 70, 96, 3
    w = wl.ksplit(M=M, K=K, N=N, P=P)
    w.out_map = (-1, 0) if scatter else (-1, -1)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=8, out_dtype=out_dtype, share_replicas=False)
    cols = st.out[0][3][-1]
    for pid, ld in enumerate(((cols + 7) // 8 * 8, cols, cols + 5)):
        t = torch.full((M * ld,), float("nan"), dtype=st.out[pid][1].dtype, device="cuda")
        st.out[pid] = (g.ShardBuf.of(t, ld), t, ld, st.out[pid][3])
    with pinned(one_launch=0):
        st.run_grouped(epilogue=1)
        assert last()[2] == 0
    ref = np.maximum(od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract), 0)
    for pid in range(P):
        want = od.expected_out_shard(ref, w.mesh_shape, w.device_ids, w.out_map, pid)
        if out_dtype == "bf16":
            want = torch.from_numpy(want).to(torch.bfloat16).double().numpy()
        assert np.array_equal(st.out_shard(pid), want), f"partition {pid}"
        _, t, ld, _ = st.out[pid]
        assert bool(torch.isnan(t.view(M, ld)[:, cols:]).all()), f"partition {pid}: beyond its rows"
