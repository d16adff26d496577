"""dot_split_kernel in tiles of 32 columns, pinned (csrc/testing.h): the sizes of its 64-column tiles' tests, and columns around 32."""
import pytest

from tests import test_gpu_kernel_edges as edges
from tests import test_gpu_split as split
from tests import test_gpu_unaligned as unaligned
from tests.pin import SPLIT, last, last_col_blocks, pinned

pytestmark = pytest.mark.gpu

SIZES = edges.SPLIT_SIZES + [(17, 640, 31), (33, 257, 32), (16, 2050, 33), (40, 96, 97)]


@pytest.mark.parametrize("row_blocks", [1, 2])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", SIZES)
def test_padded_rows(M, K, N, layout, row_blocks):
    with pinned(SPLIT, row_blocks, col_blocks=2):
        split.test_few_rows_exact(M, K, N, layout)
        assert last() == (SPLIT, row_blocks, 0) and last_col_blocks() == 2


@pytest.mark.parametrize("row_blocks", [1, 2])
@pytest.mark.parametrize("layout", [0, 1, 2, 3])
@pytest.mark.parametrize("M,K,N", unaligned.SIZES + [(40, 300, 31), (100, 77, 33), (31, 900, 59)])
def test_dense_rows_of_any_width(M, K, N, layout, row_blocks):
    with pinned(SPLIT, row_blocks, col_blocks=2):
        unaligned.test_dense_rows_of_any_width(M, K, N, 1, layout, False)
        assert last() == (SPLIT, row_blocks, 0) and last_col_blocks() == 2


@pytest.mark.parametrize("row_blocks", [1, 2])
@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_cols", [72, 261])
def test_tall_static_blocks(n_cols, out_dtype, row_blocks):
    with pinned(SPLIT, row_blocks, col_blocks=2):
        split.test_few_rows_of_tall_static_blocks(out_dtype, n_cols)
        assert last() == (SPLIT, row_blocks, 0) and last_col_blocks() == 2
