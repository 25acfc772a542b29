"""Tiles of seven column blocks (112 columns), which take one round of workgroups up to 256 x 7 blocks x K ranges of up to 64 rows, and of
eight right behind that line: whole and partial last tiles, one row and a full row tile, few and many stages, ranges of K."""
import pytest

from tests.test_gemm_tiles import test_plain_forms as check_plain, test_swiglu_forms as check_swiglu

pytestmark = pytest.mark.gpu
# (rows, columns of W / 16, K, blocks of a tile, K ranges): 1792 blocks over the whole K are 256 tiles of seven, 1793 need eight
SHAPES = [(17, 1792, 128, 7, 1), (32, 1787, 640, 7, 1), (33, 1786, 128, 7, 1), (64, 1792, 640, 7, 1), (50, 1788, 2176, 7, 1),
          (64, 1793, 128, 8, 1), (17, 1800, 640, 8, 1), (40, 2048, 640, 8, 1), (9, 896, 640, 7, 2), (16, 893, 2176, 7, 2),
          (64, 895, 2176, 7, 2), (17, 897, 2176, 8, 2), (1, 447, 2176, 7, 4), (32, 446, 4096, 7, 4), (33, 444, 2176, 7, 4),
          (64, 449, 2176, 8, 4), (9, 224, 4096, 7, 8), (64, 222, 4096, 7, 8), (33, 225, 4096, 8, 8)]


@pytest.mark.parametrize("M,blocks,K,tile,ranges", SHAPES)
def test_column_blocks(M, blocks, K, tile, ranges):
    rb = (M + 31) // 32
    check_plain(M, 16 * blocks, K, rb, tile / 2, 1, K // 32 // ranges)
    if ranges == 1:
        f_blocks = (blocks + 3) // 4 * 4             # (F % 32 == 0)
        check_swiglu(M, 8 * f_blocks, K, rb, tile / 2, 1, K // 32)
