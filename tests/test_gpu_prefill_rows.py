"""GPU parity of the column sweep whose blocks take all text rows of 32 keys (prompts of up to 64): one and two text blocks with
prompts that leave one or both empty, more samples than a wave has lanes, fewer heads than waves and numbers that eight waves do
not share evenly, one round of blocks and several, one key chunk and several, K by plain and by streaming loads.  That every call takes
this form is checked without a GPU (test_prefill_plan)."""
import pytest

import test_gpu_prefill_tiles as tiles

pytestmark = pytest.mark.gpu

SHAPES = [                                               # B, Mv, N, H, d, head_major, mask
    (5, 930, 64, 9, 128, False, True), (6, 800, 33, 3, 128, True, True), (2, 2400, 64, 20, 64, False, True), (1, 4700, 40, 17, 128, False, False),
    (70, 90, 40, 2, 64, False, True), (66, 33, 5, 12, 128, False, True), (65, 96, 64, 1, 128, False, False),     # more than 64 samples
    (24, 1190, 64, 16, 128, False, True), (24, 1190, 31, 23, 64, True, True), (18, 1500, 50, 16, 64, False, False),  # several rounds
    (9, 1000, 20, 32, 128, False, True), (2, 4640, 64, 32, 128, True, True), (9, 2000, 60, 32, 64, False, True)]     # 74 to 76 MB of K


@pytest.mark.parametrize("B,Mv,N,H,d,head_major,mask", SHAPES)
@pytest.mark.parametrize("with_lse", [False, True])
def test_all_text_rows_of_a_tile(B, Mv, N, H, d, head_major, mask, with_lse):
    tiles.test_single_tiles(B, Mv, N, H, d, head_major, mask, with_lse)
