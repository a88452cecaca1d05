"""GPU parity of the column sweep by single tiles (small calls) at its edges and around the line where the persistent form takes
over: key tiles that are not full or wholly invalid, one to four text blocks and prompts that leave some of them empty,
heads that eight waves do not share evenly, one key chunk and several, both head sizes and layouts, row normalisers."""
import numpy as np
import pytest

import oracle
import workloads as wl
from oracle import FILTER_BUDGET, FILTER_THRESHOLD
from parity import check_prefill
from test_gpu_prefill_few_rows import normalisers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Mv,N,H,d,head_major,mask", [
    (1, 1, 1, 1, 64, False, False), (2, 31, 33, 3, 128, False, True), (3, 32, 64, 8, 64, True, True), (2, 33, 65, 9, 128, True, False),
    (1, 575, 128, 20, 64, False, True), (4, 130, 97, 7, 128, False, True), (1, 2049, 32, 4, 128, False, True), (2, 700, 100, 2, 64, True, False),
    (16, 1024, 3, 2, 64, False, True), (16, 1025, 30, 2, 128, False, True), (128, 33, 127, 1, 64, False, True), (129, 33, 127, 1, 64, False, False),
    (1, 8192, 33, 2, 128, False, True), (1, 8193, 5, 2, 128, False, True),
    (1, 200, 40, 96, 64, False, True), (3, 150, 97, 96, 64, True, True), (1, 65, 7, 128, 128, False, False)])   # many heads
@pytest.mark.parametrize("with_lse", [False, True])
def test_single_tiles(B, Mv, N, H, d, head_major, mask, with_lse):
    import paper_2411_10803_amd as md
    from paper_2411_10803_amd import harness
    cfg = wl.tiny(wl.CONFIGS[2], B=B, T=1, Hg=1, Wg=Mv, N=N, H=H, d=d, C=8)
    t = wl.prefill_inputs(cfg)
    rng = np.random.default_rng(Mv * N)
    vis = (rng.random((B, Mv)) > 0.2).astype(np.uint8) if mask else None
    if mask and Mv > 64:
        vis[0, 32:64] = 0                                                        # a tile without a valid key
        vis[-1, Mv // 2:] = 0                                                    # tiles behind the last valid one
    txt_len = rng.integers(0, N + 1, size=B).astype(np.int32) if B % 2 == 0 else None
    mode = FILTER_THRESHOLD if B == 3 else FILTER_BUDGET
    R = Mv if mode == FILTER_THRESHOLD else max(1, Mv // 3)
    scale, gamma, alpha = 1.0 / np.sqrt(d), 1.0 / Mv, 2.0 / (Mv + N)
    lse = normalisers(t, Mv, np.ones((B, Mv), np.uint8) if vis is None else vis, scale) if with_lse else None
    budget = 0 if mode == FILTER_THRESHOLD else R
    print(f"B={B} Mv={Mv} N={N} H={H} d={d} head_major={head_major} mask={mask} lse={with_lse}", flush=True)
    q, k, v, hidden = (harness.to_dev(t[n], True) for n in ("q_txt", "k", "v", "hidden"))
    if head_major:
        import torch
        q, k, v = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, k, v))
        new = lambda *s, dt=torch.bfloat16: torch.zeros(s, dtype=dt, device="cuda")  # noqa: E731
        out = {"hidden_out": new(B, R + N, cfg.C), "k_out": new(B, R + N, H, d), "v_out": new(B, R + N, H, d),
               "kept_index": new(B, R, dt=torch.int32), "kept_count": new(B, dt=torch.int32), "out_len": new(B, dt=torch.int32),
               "out_protect": new(B, R + N, dt=torch.uint8), "out_ids": new(B, R + N, dt=torch.int32),
               "score_global": new(B, Mv, dt=torch.float32), "score_indiv": new(B, Mv, dt=torch.float32)}
        md.mustdrop_prefill_filter_strided(q, k, v, hidden, harness.to_dev(vis), harness.to_dev(txt_len), None, Mv, scale, mode, budget,
                                           gamma, alpha, out, Rcap=R, row_lse=harness.to_dev(lse))
    else:
        out = md.mustdrop_prefill_filter(q, k, v, hidden, harness.to_dev(vis), harness.to_dev(txt_len), None, Mv, scale, mode, budget,
                                         gamma, alpha, Rcap=R, row_lse=harness.to_dev(lse))
    g = harness.outputs_to_host(out)
    o = oracle.prefill_filter(t["q_txt"], t["k"], t["v"], t["hidden"], vis, txt_len, None, Mv, scale, mode, budget, gamma, alpha, R)
    check_prefill(g, o, t, Mv, vis, None, mode, budget, gamma, alpha, R)


# a key whose K row is no number in one head: its V is none either, and the maximum over scores that are none is 0, in both forms
# of the sweep (more than 8192 slots: the persistent one)
@pytest.mark.parametrize("B,side", [(1, 24), (3, 24), (30, 24), (1, 91)])
@pytest.mark.parametrize("with_lse", [False, True])
def test_key_row_that_is_no_number(B, side, with_lse):
    from paper_2411_10803_amd import harness
    cfg = wl.tiny(wl.CONFIGS[2], B=B, T=1, Hg=side, Wg=side, N=32, H=3, d=128, C=8)
    t = wl.prefill_inputs(cfg)
    Mv, scale = cfg.M, 1.0 / np.sqrt(128)
    lse = normalisers(t, Mv, np.ones((B, Mv), np.uint8), scale) if with_lse else None
    call = lambda: harness.prefill_on_gpu(t, Mv, None, None, None, scale, FILTER_BUDGET, 50, 1.0 / Mv, 0.1, 50, row_lse=lse)  # noqa: E731
    usual = call()
    t["k"][0, 70, 1, 5] = 0x7FC0
    g = call()
    for n, there in (("score_global", np.nan), ("score_indiv", 0.0)):
        if with_lse:                                                             # the other keys' scores do not depend on this one
            usual[n][0, 70] = there
            np.testing.assert_array_equal(g[n], usual[n])
        else:
            np.testing.assert_array_equal(g[n][0, 70], there)
            assert np.isfinite(np.delete(g[n][0], 70)).all()
            np.testing.assert_array_equal(g[n][1:], usual[n][1:])
