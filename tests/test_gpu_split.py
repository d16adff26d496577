"""dot_split_kernel (few rows: K split over the waves of a workgroup) at the sizes where it can go wrong: edges of its
row and column tiles, K steps that do not go round the eight waves evenly, K that ends inside a step, fewer steps than
waves, more than its loads run ahead, rows of the static block to clear, padding that holds NaN.  Operands are small
integers and the output float32: every order of summation is exact, so results are compared bit for bit."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import dot as od
from tests.harness import Staged

pytestmark = pytest.mark.gpu

SIZES = [   # M, K, N
    (1, 1, 1), (1, 33, 5), (15, 255, 63), (16, 256, 64), (17, 257, 65), (32, 31, 200), (33, 520, 129), (64, 1000, 1030), (65, 96, 72),
    (100, 4100, 40), (128, 2048, 192), (200, 300, 513), (256, 768, 260), (31, 6000, 70), (2, 4096, 2056),
]


def workload(M, K, N, layout):
    """One partition, out[m, n]; layout bit 0: lhs stored [K, M], bit 1: rhs stored [N, K]."""
    return wl.DotWorkload(
        name="split", cfg=7, dtype="bf16", out_dtype="f32",
        lhs_shape=(K, M) if layout & 1 else (M, K), rhs_shape=(N, K) if layout & 2 else (K, N),
        lhs_batch=(), rhs_batch=(), lhs_contract=(0,) if layout & 1 else (1,), rhs_contract=(1,) if layout & 2 else (0,),
        mesh_shape=(1,), device_ids=(0,), lhs_map=(-1, -1), rhs_map=(-1, -1), out_map=(-1, -1))


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_few_rows_exact(M, K, N, layout):
    w = workload(M, K, N, layout)
    lhs, rhs = wl.draw_small_int_bf16(3, w.lhs_shape), wl.draw_small_int_bf16(4, w.rhs_shape)
    st = Staged(w, lhs, rhs, row_align=8, out_dtype="f32")       # row padding holds NaN
    st.run_local(0, epilogue=1)
    ref = od.dot_general(wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    assert np.array_equal(st.out_shard(0), np.maximum(ref, 0.0))
    raw = st.out[0][1].view(M, -1)                               # the gap between rows is not written
    assert bool(torch.isnan(raw[:, N:]).all())


@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_cols", [72, 261])
def test_few_rows_of_tall_static_blocks(out_dtype, n_cols):
    fills = [5, 200, 0, 17, 256]                                 # occupied slots; the rest of 1500 rows is cleared
    E, C, M = len(fills), 1500, 200
    w = wl.moe(E=E, C=C, M=M, H=n_cols)
    fill = np.array(fills, dtype=np.int64)
    lhs, rhs = wl.draw_small_int_bf16(21, w.lhs_shape), wl.draw_small_int_bf16(22, w.rhs_shape)
    for e in range(E):
        lhs[e, fills[e]:] = 0x7FC0
    st = Staged(w, lhs, rhs, row_align=8, out_dtype=out_dtype)
    st.run_grouped(fill=fill)
    lhs64 = wl.bf16_bits_to_f64(lhs)
    for e in range(E):
        lhs64[e, fills[e]:] = 0.0
    ref = od.dot_general(lhs64, wl.bf16_bits_to_f64(rhs), w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    got = st.out_shard(0)
    want = ref if out_dtype == "f32" else torch.from_numpy(ref).to(torch.bfloat16).double().numpy()
    assert np.array_equal(got, want)


def test_infinities_and_nans_of_the_data_stay_where_they_are():
    w = workload(20, 100, 70, 0)
    lhs, rhs = wl.draw_small_int_bf16(5, w.lhs_shape), wl.draw_small_int_bf16(6, w.rhs_shape)
    lhs[lhs == 0] = 0x3F80                                       # no zeros: 0 x inf would be another matter
    rhs[rhs == 0] = 0x3F80
    rhs[99, 3], rhs[98, 69], lhs[7, 99] = 0x7F80, 0x7FC0, 0xFF80  # in the last K row, which a partial step holds
    st = Staged(w, lhs, rhs, row_align=8, out_dtype="f32")
    st.run_local(0)
    got = st.out_shard(0)
    a, b = wl.bf16_bits_to_f64(lhs), wl.bf16_bits_to_f64(rhs)
    with np.errstate(invalid="ignore"):
        ref = np.array([[np.sum(a[m] * b[:, n]) for n in range(70)] for m in range(20)])
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[~np.isnan(ref)], ref[~np.isnan(ref)])
