"""The edge tests of every bf16 contraction kernel on that very kernel.  A rule on sizes chooses among them, and gives most of
the small sizes at which their tiles, K steps and clears can go wrong to whichever is fastest there; here the kernel is
pinned (tests/pin.py) and every test asserts that it ran."""
import numpy as np
import pytest
import torch

import paper_2105_04663_amd as g
import workloads as wl
from oracle import dot as od
from tests import test_gpu_mid as mid
from tests import test_gpu_parity as parity
from tests import test_gpu_split as split
from tests import test_gpu_unaligned as unaligned
from tests.harness import Staged
from tests.pin import MFMA, MID, SCALAR, SPLIT, last, last_workspace, pinned

gpu = pytest.mark.gpu
ROW_BLOCKS = [1, 2, 4]


def test_pins_are_checked_and_per_thread():
    import threading
    for bad in ((4, 0, -1), (-2, 0, -1), (SPLIT, 3, -1), (SPLIT, 0, -1), (MID, 1, -1), (MFMA, 0, 2)):
        with pytest.raises(AssertionError):
            with pinned(*bad):
                pass
    seen = []
    with pinned(MID):
        t = threading.Thread(target=lambda: seen.append(last()))
        t.start()
        t.join()
    assert seen == [(-1, 0, -1)]


# --------------------------------------------------------------------------- products
# beyond the sizes of the kernel's own tests: the last tile of 32 and 64 rows or columns with 1, 8 and all but one of them, K
# beyond what the loads of a wave run ahead (4 to 6 steps of each of eight waves)
SPLIT_SIZES = split.SIZES + [(63, 300, 264), (72, 1700, 136), (129, 3000, 72), (250, 2100, 65)]


@gpu
@pytest.mark.parametrize("row_blocks", ROW_BLOCKS)
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", SPLIT_SIZES)
def test_split_kernel_padded_rows(M, K, N, layout, row_blocks):
    with pinned(SPLIT, row_blocks):
        split.test_few_rows_exact(M, K, N, layout)
        assert last() == (SPLIT, row_blocks, 0)


@gpu
@pytest.mark.parametrize("row_blocks", ROW_BLOCKS)
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_cols", [72, 261])
def test_split_kernel_tall_static_blocks(n_cols, out_dtype, row_blocks):
    with pinned(SPLIT, row_blocks):
        split.test_few_rows_of_tall_static_blocks(out_dtype, n_cols)
        assert last() == (SPLIT, row_blocks, 0)


@gpu
@pytest.mark.parametrize("kernel,row_blocks", [(SPLIT, 1), (SPLIT, 2), (SPLIT, 4), (MFMA, 0), (SCALAR, 0)])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", unaligned.SIZES)
def test_dense_rows_of_any_width(M, K, N, layout, kernel, row_blocks):
    with pinned(kernel, row_blocks):
        unaligned.test_dense_rows_of_any_width(M, K, N, 1, layout, False)
        assert last() == (kernel, row_blocks, 0)


@gpu
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N", [(259, 263), (70, 9)])
@pytest.mark.parametrize("K", [2, 7, 8, 9, 15, 16, 17, 31, 33, 39, 40, 41, 65, 71, 72, 73, 95, 97, 105])
def test_staged_tiles_that_k_ends_in(K, M, N, layout):
    # the last tile's chunks reach up to 31 positions past the valid K and are fetched from before it, below 8 element by element
    with pinned(MFMA):
        unaligned.test_dense_rows_of_any_width(M, K, N, 1, layout, False)
        assert last() == (MFMA, 0, 0)


@gpu
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("epilogue", [0, 1])
def test_staged_tiles_store_rows_of_any_width(epilogue, out_dtype):
    # shards of 301 x 177 (the last ones 300 x 177, 301 x 175), rows 187 elements apart: 16-byte stores at any element, zeros in the
    # static block's padding, nothing between the rows
    w = wl.mesh2d(M=601, K=203, N=529, X=2, Y=3, cfg=7)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=11, out_dtype=out_dtype)
    with pinned(MFMA):
        st.run_grouped(epilogue=epilogue)
        assert last() == (MFMA, 0, 0)
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    ref = np.maximum(ref, 0.0) if epilogue else ref
    if out_dtype == "bf16":
        ref = torch.from_numpy(ref).to(torch.bfloat16).double().numpy()      # integers: exact in fp32, one rounding
    for pid in range(6):
        assert np.array_equal(st.out_shard(pid), od.expected_out_shard(ref, w.mesh_shape, w.device_ids, w.out_map, pid))
        assert bool(torch.isnan(st.out[pid][1].view(301, 187)[:, 177:]).all())


@gpu
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", mid.SIZES)
def test_mid_kernel_partial_product(M, K, N, layout):
    with pinned(MID):
        mid.test_partial_product(M, K, N, layout)
        assert last() == (MID, 0, 0)


@gpu
@pytest.mark.parametrize("kernel", [MFMA, MID])
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,K,N", parity.RAGGED)
def test_ragged(M, K, N, out_dtype, kernel):
    with pinned(kernel):
        parity.test_single_partition_ragged(M, K, N, out_dtype)
        assert last() == (kernel, 0, 0)


@gpu
@pytest.mark.parametrize("kernel", [MFMA, MID])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", [(600, 200, 520), (257, 64, 255), (1, 8, 1), (513, 72, 1030), (40, 4104, 24), (260, 33, 264), (260, 95, 264),
                                   (260, 127, 264), (260, 321, 264), (470, 200, 264)])
def test_ragged_exact(M, K, N, layout, kernel):
    with pinned(kernel):
        split.test_few_rows_exact(M, K, N, layout)
        assert last() == (kernel, 0, 0)


@gpu
@pytest.mark.parametrize("kernel,row_blocks", [(MFMA, 0), (MID, 0), (SPLIT, 1), (SPLIT, 4)])
def test_fill_counts(kernel, row_blocks):
    with pinned(kernel, row_blocks):
        parity.test_fill_counts_that_end_in_every_row_block_of_a_tile()
        assert last() == (kernel, row_blocks, 0)
        for out_dtype in ("f32", "bf16"):
            parity.test_static_rows_far_below_the_last_tile_row_are_cleared(out_dtype)
            assert last() == (kernel, row_blocks, 0)
        for mode in ("local", "grouped"):
            parity.test_moe_weight_gradient_fill_limits_the_contraction(mode)
            assert last() == (kernel, row_blocks, 0)


@gpu
@pytest.mark.parametrize("kernel,row_blocks", [(MFMA, 0), (MID, 0), (SPLIT, 1), (SPLIT, 2), (SPLIT, 4)])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
def test_infinities_nans_and_denormals(layout, kernel, row_blocks):
    # K of 100: the last four positions are in a partial step; a denormal operand, a denormal sum
    w = split.workload(20, 100, 70, layout)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    lhs[lhs == 0] = 0x3F80                                       # no zeros: 0 x inf would be another matter
    rhs[rhs == 0] = 0x3F80
    a = lhs.T if layout & 1 else lhs                             # views [M, K] and [K, N]
    b = rhs.T if layout & 2 else rhs
    b[99, 3], b[98, 69], a[7, 99] = 0x7F80, 0x7FC0, 0xFF80
    a[11, :], b[:, 33] = 0x0040, 0x4980                          # 2^-127 and 2^20
    a[12, :], b[:, 34] = 0x1C80, 0x1C80                          # 2^-70 each: a sum of 100 x 2^-140
    st = Staged(w, lhs, rhs, row_align=8, out_dtype="f32")
    with pinned(kernel, row_blocks):
        st.run_local(0)
        assert last() == (kernel, row_blocks, 0)
    got = st.out_shard(0)
    with np.errstate(invalid="ignore"):
        a64, b64 = wl.bf16_bits_to_f64(np.ascontiguousarray(a)), wl.bf16_bits_to_f64(np.ascontiguousarray(b))
        ref = np.array([[np.sum(a64[m] * b64[:, n]) for n in range(70)] for m in range(20)])
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    rows, cols = [m for m in range(20) if m not in (11, 12)], [n for n in range(70) if n not in (33, 34)]
    exact = np.ix_(rows, cols)                                   # small integers and infinities
    assert np.array_equal(got[exact], ref[exact], equal_nan=True)
    assert got[11, 33] == ref[11, 33] == 100 * 2.0 ** -107 and got[12, 34] == ref[12, 34] == 100 * 2.0 ** -140


# --------------------------------------------------------------------------- sums over a contracting mesh dimension
@gpu
@pytest.mark.parametrize("kernel", [MFMA, MID])
@pytest.mark.parametrize("one_launch", [1, 0])
@pytest.mark.parametrize("M,K,N,P", [(600, 2000, 520, 4), (256, 384, 256, 3), (70, 4100, 300, 8)])
def test_sum_of_partials(M, K, N, P, one_launch, kernel):
    with pinned(kernel, 0, one_launch):
        parity.test_sum_of_partials_is_the_ascending_fp32_sum(True, M, K, N, P)
        assert last() == (kernel, 0, one_launch)


@gpu
@pytest.mark.parametrize("one_launch", [1, 0])
@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,N,P", [(300, 999, 264, 3), (129, 2048, 520, 8), (500, 70, 130, 4), (257, 33, 200, 5)])
def test_sums_of_members_by_slots(M, K, N, P, out_dtype, scatter, one_launch):
    with pinned(MFMA, 0, one_launch):
        mid.test_sums_of_members(M, K, N, P, out_dtype, scatter)
        assert last()[0] == MFMA and (scatter or last()[2] == one_launch)     # pieces of a scattered sum may not fit the workspace


@gpu
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K,N,P", [(300, 999, 264, 3), (129, 2048, 520, 8), (500, 70, 130, 4), (257, 33, 200, 5)])
def test_sums_of_members_one_after_the_other(M, K, N, P, out_dtype):
    with pinned(MID, 0, 1):
        mid.test_sums_of_members(M, K, N, P, out_dtype, False)
        assert last() == (MID, 0, 1)


@gpu
@pytest.mark.parametrize("one_launch", [1, 0])
def test_sums_of_unaligned_members(one_launch):
    # N(0, 1) data: one launch, two launches and the sum of the members' own products agree bit for bit
    w = wl.ksplit(M=300, K=199, N=201, P=3)
    lhs, rhs = wl.draw_normal_bf16(5, w.lhs_shape), wl.draw_normal_bf16(6, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=0, out_dtype="f32")
    total = None
    for pid in range(3):
        tmp = torch.full((300 * 201,), float("nan"), device="cuda")
        st.run_local(pid, out_override=g.ShardBuf.of(tmp))
        total = tmp if total is None else total + tmp
    with pinned(MFMA, 0, one_launch):
        st.run_grouped()
        assert last() == (MFMA, 0, one_launch)
    torch.cuda.synchronize()
    assert torch.equal(st.out[0][1][:300 * 201], total)
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    parity.check(st.out_shard(0), ref)


@gpu
@pytest.mark.parametrize("row_align", [8, 0])
def test_sum_over_more_members_than_the_sum_kernels_take(row_align):
    # 40 partitions share 5 positions of K: 35 of them have nothing to add, and only the one-launch sum can leave them out
    w = wl.ksplit(M=70, K=5, N=75, P=40)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=row_align, out_dtype="f32")
    st.run_grouped()
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    assert np.array_equal(st.out_shard(0), ref)


@gpu
@pytest.mark.parametrize("M,K,N,P,row_align,one_launch", [(141, 7248, 463, 8, 8, 0), (659, 4880, 1316, 2, 8, 0), (727, 205, 74, 8, 0, 0),
                                                          (1953, 409, 454, 4, 8, 1), (4023, 8430, 1215, 8, 8, 1),
                                                          (1335, 508, 4085, 2, 0, 1)])
def test_sums_take_the_way_that_measured_faster(M, K, N, P, row_align, one_launch):
    # sizes at which one way took at most 0.9 of the other's time when the rule was made, by its estimates too
    w = wl.ksplit(M=M, K=K, N=N, P=P)
    st = Staged(w, np.zeros(w.lhs_shape, dtype=np.uint16), np.zeros(w.rhs_shape, dtype=np.uint16), row_align=row_align)
    st.run_grouped()
    assert last()[2] == one_launch


@gpu
@pytest.mark.parametrize("kernel", [MFMA, MID])
@pytest.mark.parametrize("row_align", [8, 0])
@pytest.mark.parametrize("M,K,N,P", [(257, 520, 320, 8), (300, 999, 2051, 6), (70, 1000, 4096, 16)])
def test_scattered_sums_whose_tables_are_uploaded(M, K, N, P, row_align, kernel):
    # more pieces than travel as kernel arguments, and a workspace with room for their table beside counters and slots
    w = wl.ksplit(M=M, K=K, N=N, P=P)
    w.out_map = (-1, 0)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=row_align, out_dtype="f32")
    n = g.dot_workspace_bytes(st.mesh, st.dims, st.lhs_sh, st.rhs_sh, st.out_sh) + P * P * -(-M // 256) * -(-N // (256 * P)) * 270 * 1024
    ws = torch.full((n + 256,), 255, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    for rep in range(3):
        for _, t, _, _ in st.out:
            t.fill_(float("nan"))
        with pinned(kernel, 0, 1):
            g.grouped_dot(st.mesh, st.dims, [x[0] for x in st.lhs], st.lhs_sh, [x[0] for x in st.rhs], st.rhs_sh, [x[0] for x in st.out], st.out_sh,
                          None, base, n, torch.cuda.current_stream().cuda_stream)
            assert last()[2] == 1 and last_workspace()[0] > 0
        for pid in range(P):
            assert np.array_equal(st.out_shard(pid), od.expected_out_shard(ref, w.mesh_shape, w.device_ids, w.out_map, pid)), f"rep {rep} pid {pid}"
