"""GPU parity of the wide row statistics with one block per sample and head: 65 to 128 text rows where the heads of all samples nearly
fill the CUs, and where they are more than two rounds of blocks; tiles without a valid key, prompts of fewer text blocks.
That every call takes this form is checked without a GPU (test_prefill_plan)."""
import pytest

import test_gpu_prefill_tiles as tiles

pytestmark = pytest.mark.gpu


SHAPES = [                                               # B, Mv, N, H, d, head_major, mask
    (6, 930, 100, 30, 128, False, True), (5, 905, 97, 37, 128, True, False),
    (33, 200, 70, 16, 128, True, True), (34, 130, 128, 17, 128, False, True)]


@pytest.mark.parametrize("B,Mv,N,H,d,head_major,mask", SHAPES)
def test_one_wide_block_per_head(B, Mv, N, H, d, head_major, mask):
    tiles.test_single_tiles(B, Mv, N, H, d, head_major, mask, False)
