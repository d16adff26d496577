"""Stores of whole lines (csrc/kernels_lines.h) at the edges of a lane's 16 bytes, of a wave's 64 rows and columns and of a tile, at aligned and odd
output rows: the output's memory, the gaps between rows included, is that of dot_mfma_kernel, bit for bit."""
import pytest
import torch

import workloads as wl
from tests import test_gpu_split as split
from tests.harness import Staged
from tests.pin import MFMA, MID, PAIR, last, pinned

pytestmark = pytest.mark.gpu


def _same_memory(w, kernel, row_align, out_dtype, epilogue):
    lhs, rhs = wl.draw_normal_bf16(w.lhs_shape[0], w.lhs_shape), wl.draw_normal_bf16(w.rhs_shape[1], w.rhs_shape)
    raw = []
    for k in (kernel, MFMA):
        st = Staged(w, lhs, rhs, row_align=row_align, out_dtype=out_dtype)
        with pinned(k):
            st.run_grouped(epilogue=epilogue)
            assert last()[0] == k
        out = st.out[0][1]
        raw.append(out.view(torch.int16 if out_dtype == "bf16" else torch.int32).cpu())
    assert torch.equal(*raw)


# (operands at odd addresses, K 71 in dense rows, are not for dot_pair_kernel)
@pytest.mark.parametrize("epilogue", [0, 1])
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kernel,K,row_align", [(MID, 72, 8), (MID, 72, 0), (MID, 71, 0), (PAIR, 72, 8), (PAIR, 72, 0)])
@pytest.mark.parametrize("M,N", [(1, 1), (15, 7), (33, 8), (63, 9), (64, 64), (65, 68), (127, 63), (128, 128), (129, 130), (255, 121), (256, 129), (300, 391)])
def test_edges(M, N, kernel, K, row_align, out_dtype, epilogue):
    _same_memory(split.workload(M, K, N, 2), kernel, row_align, out_dtype, epilogue)      # both operands K-contiguous: their rows do not depend on the output's width


# Dense rows of K-major operands, where the last tiles are moved back: of both operands in dot_mid_kernel's staged tiles (odd extents), of the rhs in
# direct ones (even extents; rows of a K-major lhs are padded by their number).
@pytest.mark.parametrize("epilogue", [0, 1])
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", [0, 1, 3])
@pytest.mark.parametrize("kernel,M,K,N", [(MID, 129, 71, 131), (MID, 255, 100, 257), (MID, 391, 33, 389), (MID, 136, 72, 130), (MID, 264, 72, 390),
                                          (PAIR, 136, 72, 130), (PAIR, 264, 72, 390), (PAIR, 512, 136, 254)])
def test_tiles_that_are_moved_back(kernel, M, K, N, layout, out_dtype, epilogue):
    _same_memory(split.workload(M, K, N, layout), kernel, 0, out_dtype, epilogue)


@pytest.mark.parametrize("K", [40, 41])              # direct and staged loads
def test_outputs_that_the_caches_do_not_hold(K):
    _same_memory(split.workload(6203, K, 7801, 2), MID, 0, "bf16", 0)          # 97 MB: past the caches


def test_operands_that_take_much_of_the_caches():
    _same_memory(split.workload(391, 20000, 1402, 2), MID, 8, "bf16", 1)       # 72 MB: past the caches
