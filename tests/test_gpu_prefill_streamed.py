"""Calls of a size from which on memory is passed by the Infinity Cache.

The row statistics of a K that outgrows the Infinity Cache, read by streaming loads: every form that has them (one and two text
blocks, the wide one) and heads of 64, which do not, with tiles that are not full, masks and prompts that leave text blocks empty.  The
column sweep of several text groups where their query fragments are 28 MB and more.  The copies of head-major rows where K is more than
100 MB, with the K rows out by streaming stores and, with the caller's normalisers, by plain ones."""
import pytest

import test_gpu_prefill_tiles as tiles
from test_gpu_prefill_wide import test_row_statistics as row_statistics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Mv,N,H,d,mask,txt", [
    (3, 18500, 32, 32, 128, "holes", [32, 5, 20]), (8, 9161, 30, 33, 64, None, None),                 # 455 and 310 MB, one text block
    (2, 18700, 64, 32, 128, None, [64, 31]), (8, 9200, 48, 32, 64, "prefix", None),                   # 306 and 301 MB, two
    (7, 9169, 97, 15, 128, "holes", None), (40, 1501, 70, 16, 128, "prefix", None),                   # 246 MB, the wide form
    (7, 9172, 113, 29, 64, "holes", [113, 97, 64, 33, 32, 1, 80])])                                   # 238 MB, four
def test_streamed_row_statistics(B, Mv, N, H, d, mask, txt):
    row_statistics(B, Mv, N, H, d, mask, txt)


@pytest.mark.parametrize("B,Mv,N,H,d,with_lse", [(13, 70, 257, 32, 128, False), (13, 70, 257, 32, 128, True), (26, 65, 257, 32, 64, False)])
def test_column_sweep_of_many_fragments(B, Mv, N, H, d, with_lse):
    assert B * H * d * 2 * 32 * 9 >= 28e6
    tiles.test_single_tiles(B, Mv, N, H, d, False, True, with_lse)


@pytest.mark.parametrize("with_lse", [False, True])
def test_copies_of_large_head_major_calls(with_lse):
    B, Mv, N, H, d = 4, 3000, 20, 34, 128
    assert B * (Mv + N) * H * d * 2 > 100e6
    tiles.test_single_tiles(B, Mv, N, H, d, True, True, with_lse)
