"""The row statistics of a K that outgrows the Infinity Cache, read by streaming loads: every form that has them (one, two and four text
blocks, the wide one, heads of 64), with tiles that are not full, masks and prompts that leave text blocks empty."""
import pytest

from test_gpu_prefill_wide import test_row_statistics as row_statistics

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Mv,N,H,d,mask,txt", [
    (2, 18500, 32, 32, 128, "holes", [32, 5]), (8, 9161, 30, 33, 64, None, None),                     # 303 and 310 MB, one text block
    (2, 18700, 64, 32, 128, None, [64, 31]), (8, 9200, 48, 32, 64, "prefix", None),                   # 306 and 301 MB, two
    (7, 9169, 97, 15, 128, "holes", None), (40, 1501, 70, 16, 128, "prefix", None),                   # 246 MB, the wide form
    (7, 9172, 113, 29, 64, "holes", [113, 97, 64, 33, 32, 1, 80])])                                   # 238 MB, four
def test_streamed_row_statistics(B, Mv, N, H, d, mask, txt):
    row_statistics(B, Mv, N, H, d, mask, txt)
