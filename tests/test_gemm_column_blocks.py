"""Tiles of seven column blocks (112 columns), which take one round of workgroups up to 256 x 7 blocks of up to 64 rows, and of eight
right behind that line: whole and partial last tiles, one row and a full row tile, few and many stages."""
import pytest

from tests.test_gemm_tiles import test_plain_forms as check_plain, test_swiglu_forms as check_swiglu

pytestmark = pytest.mark.gpu
# (rows, columns of W / 16, K): 1792 blocks are 256 tiles of seven, 1793 need eight
SHAPES = [(17, 1792, 128), (32, 1787, 640), (33, 1786, 128), (64, 1792, 640), (50, 1788, 2176), (64, 1793, 128), (17, 1800, 640),
          (40, 2048, 640)]


@pytest.mark.parametrize("M,blocks,K", SHAPES)
def test_column_blocks(M, blocks, K):
    rb = (M + 31) // 32
    check_plain(M, 16 * blocks, K, rb, 4, 1, K // 32)
    f_blocks = (blocks + 3) // 4 * 4                 # (F % 32 == 0)
    check_swiglu(M, 8 * f_blocks, K, rb, 4, 1, K // 32)
