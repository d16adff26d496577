"""dot_pair_kernel pinned (csrc/testing.h) at the edges of its tiles of 256 x 128, its ring of three 32-wide K tiles and its unrolled loop of six: small
integers, compared exactly; bit for bit with dot_mfma_kernel on random values; loose rows; blocks to be cleared."""
import numpy as np
import pytest

import workloads as wl
from tests import test_gpu_parity as parity
from tests import test_gpu_split as split
from tests import test_gpu_word_rows as words
from tests.harness import Staged
from tests.pin import MFMA, PAIR, last, pinned

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", [(257, 64, 129), (1, 8, 1), (513, 72, 1030), (40, 4104, 24), (256, 32, 128), (255, 31, 127), (600, 1, 520), (129, 40, 260)] +
                         [(300, k, 140) for k in (33, 65, 96, 97, 127, 128, 160, 200, 224, 255, 256, 288, 289, 300, 319, 320, 321, 480, 511, 512)])
def test_tiles_and_k(M, K, N, layout):
    with pinned(PAIR):
        split.test_few_rows_exact(M, K, N, layout)
        assert last() == (PAIR, 0, 0)


@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,K,N", parity.RAGGED)
def test_ragged(M, K, N, out_dtype):
    with pinned(PAIR):
        parity.test_single_partition_ragged(M, K, N, out_dtype)
        assert last() == (PAIR, 0, 0)


def test_fill_counts():
    with pinned(PAIR):
        parity.test_fill_counts_that_end_in_every_row_block_of_a_tile()
        assert last() == (PAIR, 0, 0)
        for out_dtype in ("f32", "bf16"):
            parity.test_static_rows_far_below_the_last_tile_row_are_cleared(out_dtype)
            assert last() == (PAIR, 0, 0)
        for mode in ("local", "grouped"):
            parity.test_moe_weight_gradient_fill_limits_the_contraction(mode)
            assert last() == (PAIR, 0, 0)


@pytest.mark.parametrize("epilogue", [0, 1])
@pytest.mark.parametrize("out_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
def test_same_bits_as_the_large_tiles(layout, out_dtype, epilogue):
    w = split.workload(777, 329, 1033, layout)
    lhs, rhs = wl.draw_normal_bf16(layout, w.lhs_shape), wl.draw_normal_bf16(layout + 4, w.rhs_shape)
    got = []
    for kernel in (PAIR, MFMA):
        st = Staged(w, lhs, rhs, row_align=8, out_dtype=out_dtype)
        with pinned(kernel):
            st.run_grouped(epilogue=epilogue)
            assert last() == (kernel, 0, 0)
        got.append(st.out_shard(0))
    assert np.array_equal(*got)


@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N,Y", [(256, 64, 256, 1), (304, 104, 257, 1), (40, 72, 511, 1), (520, 200, 770, 1), (264, 320, 3 * 300 - 4, 3), (128, 8, 129, 1)])
def test_rows_of_whole_words(M, K, N, Y, layout):
    words.test_products(M, K, N, Y, layout, PAIR)


@pytest.mark.parametrize("H", [300, 301, 512, 770])
@pytest.mark.parametrize("fill", [(10, 0, 257), (600, 17, 511)])
def test_rows_below_a_moved_tile_are_cleared(H, fill, monkeypatch):
    monkeypatch.setattr(words, "MFMA", PAIR)                         # the kernel that the test pins and asks for
    words.test_rows_below_a_moved_tile_are_cleared(H, fill)
