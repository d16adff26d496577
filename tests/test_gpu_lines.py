"""Stores of whole lines (csrc/kernels_lines.h) at the edges of a lane's 16 bytes, of a wave's 64 rows and columns and of a tile, at aligned and odd
output rows: the output's memory, the gaps between rows included, is that of dot_mfma_kernel, bit for bit."""
import pytest
import torch

import workloads as wl
from tests import test_gpu_split as split
from tests.harness import Staged
from tests.pin import MFMA, MID, PAIR, last, pinned

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("epilogue", [0, 1])
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("K,row_align", [(72, 8), (72, 0), (71, 0)])
@pytest.mark.parametrize("kernel", [MID, PAIR])
@pytest.mark.parametrize("M,N", [(1, 1), (15, 7), (33, 8), (63, 9), (64, 64), (65, 68), (127, 63), (128, 128), (129, 130), (255, 121), (256, 129), (300, 391)])
def test_edges(M, N, kernel, K, row_align, out_dtype, epilogue):
    if kernel == PAIR and K % 2:
        pytest.skip("operands at odd addresses are not for this kernel")
    w = split.workload(M, K, N, 2)                  # both operands K-contiguous: their rows do not depend on the output's width
    lhs, rhs = wl.draw_normal_bf16(M, w.lhs_shape), wl.draw_normal_bf16(N, w.rhs_shape)
    raw = []
    for k in (kernel, MFMA):
        st = Staged(w, lhs, rhs, row_align=row_align, out_dtype=out_dtype)
        with pinned(k):
            st.run_grouped(epilogue=epilogue)
            assert last()[0] == k
        out = st.out[0][1]
        raw.append(out.view(torch.int16 if out_dtype == "bf16" else torch.int32).cpu())
    assert torch.equal(*raw)
