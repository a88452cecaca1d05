"""GPU parity of the prefill row statistics, whose key sweep ends at each sample's txt_len: lengths at the edges of the 32-key tiles, vision
rows that fill their last tile and that do not, samples without a valid vision key, both forms of the sweep; the K and Q rows behind txt_len
are no numbers."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_prefill import run

pytestmark = pytest.mark.gpu


# one, two and four text blocks, several text groups (the wide form), heads of 64; (700, 640): more text steps than vision steps
@pytest.mark.parametrize("Mv,N,H,d", [
    (200, 32, 20, 128), (1025, 33, 20, 128), (96, 64, 20, 64), (1000, 128, 3, 128), (577, 128, 24, 128), (330, 128, 20, 64),
    (321, 300, 8, 128), (64, 300, 3, 64), (700, 640, 4, 128)])
@pytest.mark.parametrize("mask", [False, True])
def test_sweep_ends_at_text_length(Mv, N, H, d, mask):
    lens = sorted({0, 1, 31, 32, 33, N // 2, N - 1, N} & set(range(N + 1)))
    B, R = len(lens), max(1, Mv // 4)
    cfg = wl.tiny(wl.CONFIGS[2], B=B, T=1, Hg=1, Wg=Mv, N=N, H=H, d=d, C=8)
    t = wl.prefill_inputs(cfg)
    vis = None
    if mask:
        vis = (np.random.default_rng(Mv + N).random((B, Mv)) > 0.3).astype(np.uint8)
        vis[1::3, Mv // 2:] = 0                                                  # the effective rows end in the middle
        vis[2::3] = 0                                                            # none at all
    for b, n in enumerate(lens):
        t["k"][b, Mv + n:] = 0x7FC0
        t["q_txt"][b, n:] = 0x7FC0
    print(f"Mv={Mv} N={N} H={H} d={d} mask={mask} lens={lens}", flush=True)
    run(t, Mv, R, vis_valid=vis, txt_len=np.array(lens, np.int32))
