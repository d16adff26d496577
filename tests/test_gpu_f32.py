"""dot_f32_kernel at the edges of its tiles and K steps, in all four operand layouts, dense and padded rows: small
integers (exact, compared bit for bit), and random values against float64 with the bound of a float32 sum:
|error| <= (K + 2) * 2^-24 * sum |a b| for any order of summation."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import dot as od
from tests.harness import Staged
from tests.test_gpu_split import workload

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (3, 31, 5), (64, 32, 64), (65, 33, 63), (63, 64, 65), (8, 64, 23), (130, 100, 67), (200, 5, 129), (128, 257, 192), (70, 1000, 300)]


@pytest.mark.parametrize("align", [0, 8])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_f32_tiles(M, K, N, layout, align):
    w = workload(M, K, N, layout)
    w.dtype = "f32"
    rng = np.random.default_rng(5)
    for exact in (True, False):
        if exact:
            lhs, rhs = (rng.integers(-50, 51, size=s).astype(np.float32) for s in (w.lhs_shape, w.rhs_shape))
        else:
            lhs, rhs = (rng.uniform(-1, 1, size=s).astype(np.float32) for s in (w.lhs_shape, w.rhs_shape))
        st = Staged(w, lhs, rhs, row_align=align)                # row padding holds NaN
        st.run_local(0)
        got = st.out_shard(0)
        dims = (w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
        a, b = lhs.astype(np.float64), rhs.astype(np.float64)
        ref = od.dot_general(a, b, *dims)
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert (np.abs(got - ref) <= (K + 2) * 2.0 ** -24 * od.dot_general(np.abs(a), np.abs(b), *dims)).all()
        if align and N % 8:
            assert bool(torch.isnan(st.out[0][1].view(M, -1)[:, N:]).all())


def test_f32_special_values():
    # infinities and NaNs of the data reach exactly the outputs they belong to; denormal products and operands are kept
    w = workload(20, 37, 40, 0)
    w.dtype = "f32"
    lhs, rhs = np.ones(w.lhs_shape, np.float32), np.ones(w.rhs_shape, np.float32)
    rhs[36, 3], rhs[0, 39], lhs[7, 36] = np.inf, np.nan, -np.inf
    st = Staged(w, lhs, rhs, row_align=8)
    st.run_local(0)
    got = st.out_shard(0)
    with np.errstate(invalid="ignore"):
        ref = np.array([[np.sum(lhs[m].astype(np.float64) * rhs[:, n].astype(np.float64)) for n in range(40)] for m in range(20)])
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[~np.isnan(ref)], ref[~np.isnan(ref)])
    tiny = np.float32(2.0 ** -140)
    lhs, rhs = np.zeros(w.lhs_shape, np.float32), np.zeros(w.rhs_shape, np.float32)
    lhs[:, 0], rhs[0, :] = tiny, 1.0
    lhs[:, 1], rhs[1, :] = 2.0 ** -70, 2.0 ** -75
    st = Staged(w, lhs, rhs, row_align=8)
    st.run_local(0)
    assert (st.out_shard(0) == float(tiny) + 2.0 ** -145).all()


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", [(2001, 37, 2030), (2501, 70, 2390)])          # 1024 tiles: four workgroups on a compute unit; 1520: three
def test_f32_workgroups_on_a_compute_unit(M, K, N, layout):
    w = workload(M, K, N, layout)
    w.dtype = "f32"
    rng = np.random.default_rng(5)
    lhs, rhs = (rng.integers(-50, 51, size=s).astype(np.float32) for s in (w.lhs_shape, w.rhs_shape))
    st = Staged(w, lhs, rhs, row_align=0)
    st.run_local(0)
    dims = (w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    assert np.array_equal(st.out_shard(0), od.dot_general(lhs.astype(np.float64), rhs.astype(np.float64), *dims))


# K steps around the stages' count and the unrolled loop (three and two stages), with a part of a step left or not; columns that end inside a chunk
@pytest.mark.parametrize("layout", [0, 3])
@pytest.mark.parametrize("M,N", [(66, 129), (1985, 2047)])          # 6 tiles; 1024: four workgroups on a compute unit
@pytest.mark.parametrize("K", [96, 128, 130, 160, 192, 224, 255, 288])
def test_f32_steps(M, N, K, layout):
    w = workload(M, K, N, layout)
    w.dtype = "f32"
    rng = np.random.default_rng(K)
    lhs, rhs = (rng.integers(-50, 51, size=s).astype(np.float32) for s in (w.lhs_shape, w.rhs_shape))
    st = Staged(w, lhs, rhs, row_align=0)
    st.run_local(0)
    dims = (w.lhs_batch, w.rhs_batch, w.lhs_contract, w.rhs_contract)
    assert np.array_equal(st.out_shard(0), od.dot_general(lhs.astype(np.float64), rhs.astype(np.float64), *dims))


def test_f32_rows_beyond_32_bit_offsets():
    import paper_2105_04663_amd as g
    stride, M, K, N = 1 << 27, 3, 70, 9                              # rows of 512 MiB
    rng = np.random.default_rng(1)
    lhs, rhs = rng.integers(-50, 51, size=(M, K)).astype(np.float32), rng.integers(-50, 51, size=(K, N)).astype(np.float32)
    a = torch.empty((M - 1) * stride + K, dtype=torch.float32, device="cuda")
    for m in range(M):
        a[m * stride:m * stride + K] = torch.from_numpy(lhs[m])
    b, out = torch.from_numpy(rhs).cuda(), torch.empty(M, N, dtype=torch.float32, device="cuda")
    mesh, dims = g.Mesh((1,), (0,)), g.DotDims((), (), (1,), (0,))
    lsh, rsh, osh = (g.Sharding(s, (-1, -1)) for s in ((M, K), (K, N), (M, N)))
    ws = torch.empty(g.dot_workspace_bytes(mesh, dims, lsh, rsh, osh, 0, False) + 256, dtype=torch.uint8, device="cuda")
    g.local_dot(mesh, dims, g.ShardBuf(a.data_ptr(), g.F32, stride), lsh, g.ShardBuf(b.data_ptr(), g.F32, 0), rsh, g.ShardBuf(out.data_ptr(), g.F32, 0), osh,
                0, None, (ws.data_ptr() + 255) // 256 * 256, ws.numel() - 256, torch.cuda.current_stream().cuda_stream)
    assert np.array_equal(out.cpu().numpy(), lhs.astype(np.float64) @ rhs.astype(np.float64))


def _wide(M, K, N, layout, wide):
    """A float32 product on one device with the rows of one operand (`wide`: "lhs", "rhs") 2^27 elements apart; as a call, its output and its operands."""
    import paper_2105_04663_amd as g
    shapes = {"lhs": (K, M) if layout & 1 else (M, K), "rhs": (N, K) if layout & 2 else (K, N)}
    keep, bufs = [], {}
    gen = torch.Generator(device="cuda").manual_seed(3)
    values = {}
    for name, (rows, cols) in shapes.items():
        stride = 1 << 27 if name == wide else cols
        store = torch.empty((rows - 1) * stride + cols, dtype=torch.float32, device="cuda")
        values[name] = torch.randint(-50, 51, (rows, cols), generator=gen, device="cuda").float()
        store.as_strided((rows, cols), (stride, 1)).copy_(values[name])
        keep.append(store)
        bufs[name] = g.ShardBuf(store.data_ptr(), g.F32, stride)
    out = torch.empty(M, N, dtype=torch.float32, device="cuda")
    mesh, dims = g.Mesh((1,), (0,)), g.DotDims((), (), (0 if layout & 1 else 1,), (1 if layout & 2 else 0,))
    lsh, rsh, osh = (g.Sharding(s, (-1, -1)) for s in (shapes["lhs"], shapes["rhs"], (M, N)))
    ws = torch.empty(g.dot_workspace_bytes(mesh, dims, lsh, rsh, osh, 0, False) + 256, dtype=torch.uint8, device="cuda")

    def run():
        g.local_dot(mesh, dims, bufs["lhs"], lsh, bufs["rhs"], rsh, g.ShardBuf(out.data_ptr(), g.F32, 0), osh, 0, None, (ws.data_ptr() + 255) // 256 * 256, ws.numel() - 256,
                    torch.cuda.current_stream().cuda_stream)
    run.keep = keep, ws
    return run, out, values


# 66 wide rows: two tiles of them, or two K steps and two rows left; columns that end inside a chunk
@pytest.mark.parametrize("M,K,N,layout,wide", [(66, 230, 131, 0, "lhs"), (131, 66, 70, 1, "lhs"), (70, 66, 131, 0, "rhs"), (131, 230, 66, 2, "rhs"), (70, 66, 131, 3, "lhs"), (3, 66, 131, 3, "lhs")])
def test_f32_rows_beyond_32_bit_offsets_in_every_layout(M, K, N, layout, wide):
    run, out, v = _wide(M, K, N, layout, wide)
    run()
    a, b = (v["lhs"].T if layout & 1 else v["lhs"]).double().cpu(), (v["rhs"].T if layout & 2 else v["rhs"]).double().cpu()
    assert torch.equal(out.double().cpu(), a @ b)                    # whole numbers below 2^24: every sum is exact


def test_f32_rows_beyond_32_bit_offsets_at_full_speed():
    """Within twice the time of rows that are near each other (measured 1.1 times; loads element by element 3.5 times)."""
    least = {}
    for wide in (None, "lhs"):
        run, _, _ = _wide(64, 2048, 8192, 0, wide)
        times = []
        for _ in range(6):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(20):
                run()
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end))
        least[wide] = min(times)
    assert least["lhs"] < 2 * least[None], least
