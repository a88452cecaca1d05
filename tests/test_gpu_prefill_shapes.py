"""GPU parity of the score sweeps where their launch shapes change: several text groups with prompts of any length down
to none, wave columns without text rows, blocks of four and eight waves, several key chunks, streaming loads."""
import numpy as np
import pytest

import workloads as wl
from oracle import FILTER_BUDGET, FILTER_THRESHOLD
from test_gpu_prefill import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hg,Wg,N,H,d,txt", [
    (9, 13, 129, 3, 128, [129, 0, 33]),              # two groups; one sample has none, one a single block
    (20, 20, 260, 2, 64, [1, 260, 128, 129]),        # three groups of three; the others one, one and two
    (6, 5, 384, 5, 128, None),
    (30, 31, 300, 2, 128, [300, 97]),
    (7, 7, 1024, 1, 64, [1024, 700]),                # eight groups
    (25, 24, 65, 4, 128, [65, 64]),                  # three blocks of text rows in four wave columns
    (24, 25, 20, 64, 64, None),                      # 1 x 8 waves
    (18, 43, 60, 16, 128, [60, 31, 32, 33, 1]),      # 2 x 4 waves
    (60, 60, 100, 4, 64, [100, 0]),                  # several key chunks, an empty prompt
])
@pytest.mark.parametrize("padded", [False, True])
def test_launch_shapes(Hg, Wg, N, H, d, txt, padded):
    cfg = wl.tiny(wl.CONFIGS[2], B=len(txt) if txt else 2, T=1, Hg=Hg, Wg=Wg, N=N, H=H, d=d, C=72)
    Mv = cfg.M
    t = wl.prefill_inputs(cfg)
    rng = np.random.default_rng(Mv + N)
    vis = None
    if padded:
        vis = np.zeros((cfg.B, Mv), np.uint8)
        for b in range(cfg.B):
            vis[b, :rng.integers(1, Mv + 1)] = 1
    txt_len = None if txt is None else np.array(txt, np.int32)
    is_key = wl.random_key_mask(cfg, min(8, Mv // 4), valid=vis)
    R = max(Mv // 3, int(is_key.sum(1).max()))
    run(t, Mv, R, vis_valid=vis, txt_len=txt_len, is_key=is_key)
    run(t, Mv, 0, mode=FILTER_THRESHOLD, vis_valid=vis, txt_len=txt_len, is_key=is_key, alpha=1.2 / (Mv + N), Rcap=Mv)


@pytest.mark.parametrize("N", [3, 40])
def test_keys_beyond_the_infinity_cache(N):
    cfg = wl.tiny(wl.CONFIGS[2], B=1, T=1, Hg=140, Wg=144, N=N, H=32, d=128, C=64)
    t = wl.prefill_inputs(cfg)
    run(t, cfg.M, 500, mode=FILTER_BUDGET, is_key=wl.random_key_mask(cfg, 50))


def test_row_normalisers_with_several_text_groups():
    from paper_2411_10803_amd import harness
    import oracle
    cfg = wl.tiny(wl.CONFIGS[2], B=3, T=1, Hg=17, Wg=19, N=290, H=3, d=128, C=64)
    Mv, L, txt_len = cfg.M, cfg.M + cfg.N, np.array([290, 60, 130], np.int32)
    t = wl.prefill_inputs(cfg)
    q, k = (wl.bf16_bits_to_f32(t[n]).astype(np.float64) for n in ("q_txt", "k"))
    scale = 1.0 / np.sqrt(128)
    s = np.einsum("bihd,bjhd->bhij", q, k) * scale
    seen = np.concatenate([np.ones((cfg.N, Mv), bool), np.tril(np.ones((cfg.N, cfg.N), bool))], 1)
    s = np.where(seen, s, -np.inf)
    m = s.max(-1, keepdims=True)
    lse = (m[..., 0] + np.log(np.exp(s - m).sum(-1))).astype(np.float32)
    R, gamma, alpha = 100, 1.0 / Mv, 2.0 / L
    is_key = wl.random_key_mask(cfg, 10)
    g = harness.prefill_on_gpu(t, Mv, None, txt_len, is_key, scale, FILTER_BUDGET, R, gamma, alpha, R, row_lse=lse)
    o = oracle.prefill_filter(t["q_txt"], t["k"], t["v"], t["hidden"], None, txt_len, is_key, Mv, scale, FILTER_BUDGET, R,
                              gamma, alpha, R)
    from parity import check_prefill
    check_prefill(g, o, t, Mv, None, is_key, FILTER_BUDGET, R, gamma, alpha, R)
