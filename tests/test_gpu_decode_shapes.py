"""GPU parity of the streaming scoring and in-register selection kernels at head shapes off the powers of two: rows that
end inside a 1 KiB piece, heads in fours, both cache layouts, the steady state (one entry leaves) and large cuts, with the row
moves in the selection's launch or in their own."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import check_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d,L0,cut", [(12, 64, 130, 1), (20, 128, 1025, 1), (36, 64, 700, 300), (40, 64, 2100, 1),
                                        (40, 128, 1500, 900), (48, 128, 330, 1), (64, 128, 513, 100), (128, 64, 260, 3),
                                        (3, 128, 200, 50), (40, 128, 4100, 3000), (44, 128, 300, 1), (124, 64, 260, 90)])
@pytest.mark.parametrize("head_major", [False, True])
def test_head_shapes(H, d, L0, cut, head_major):
    check(H, d, L0, cut, head_major, None)


# a few live entries of many slots: the moves have a launch of their own, unless four rows or fewer move
@pytest.mark.parametrize("cut", [1, 4, 5, 600])
def test_long_caches_with_few_entries(cut):
    check(32, 64, 1000, cut, False, 8000)


# a cut of many rows by more than 64 blocks per sample, all teams busy and not
@pytest.mark.parametrize("H,L0,cut,slots", [(32, 2400, 1900, None), (16, 700, 520, None), (4, 5000, 4100, 8192)])
@pytest.mark.parametrize("head_major", [False, True])
def test_many_blocks_per_sample(H, L0, cut, slots, head_major):
    check(H, 64, L0, cut, head_major, slots)


# the largest LDS a selection in registers asks for
@pytest.mark.parametrize("H,slots", [(64, 8192), (96, 4096)])
@pytest.mark.parametrize("cut", [1, 200])
def test_most_lds(H, slots, cut):
    check(H, 64, 1200, cut, False, slots)


# entries that a caller masks through their keys, on all heads or on some: their logits are -inf, their probabilities zero
@pytest.mark.parametrize("H,d,L0,cut", [(40, 128, 1025, 1), (12, 64, 300, 100), (40, 64, 700, 1), (32, 128, 1025, 1),
                                        (3, 128, 200, 50), (8, 32, 400, 1)])
@pytest.mark.parametrize("head_major", [False, True])
def test_masked_entries(H, d, L0, cut, head_major):
    check(H, d, L0, cut, head_major, None, masked=True)


def check(H, d, L0, cut, head_major, slots, masked=False):
    import torch
    import paper_2411_10803_amd as md
    from paper_2411_10803_amd import harness
    budget = L0 - cut
    cfg = wl.tiny(wl.CONFIGS[5], B=2, L0=L0, steps=1, decode_budget=budget, n_protect=min(20, budget), H=H, d=d)
    t = wl.decode_inputs(cfg, Lcap=slots)
    B, Lcap = cfg.B, t["Lcap"]
    rng = np.random.default_rng(H * L0)
    s0 = {"k": t["k_cache"], "v": t["v_cache"], "acc": rng.random((B, Lcap)).astype(np.float32) * np.float32(1.0 / L0),
          "ids": np.stack([rng.permutation(2 * Lcap)[:Lcap] for _ in range(B)]).astype(np.int32),
          "protect": t["protect"].copy(), "len": t["len0"].copy()}
    if masked:
        minus_inf, plus_inf = 0xFF80, 0x7F80
        sign = t["q_steps"][0][:, :, 0] >> 15                                    # [B, H]: an infinity of the other sign than q's
        hide = rng.random((B, Lcap, H)) < 0.1
        hide[:, ::7] = True
        s0["k"][..., 0] = np.where(hide, np.where(sign[:, None] != 0, plus_inf, minus_inf), s0["k"][..., 0]).astype(np.uint16)
    scale, decay = 1.0 / np.sqrt(d), 0.75
    dv = harness.decode_state_to_dev(s0)
    q = harness.to_dev(t["q_steps"][0], True)
    ev = torch.full((B, Lcap), -1, dtype=torch.int32, device="cuda")
    evc = torch.zeros((B,), dtype=torch.int32, device="cuda")
    if head_major:
        for name in ("k", "v"):
            dv[name] = dv[name].transpose(1, 2).contiguous().transpose(1, 2)
        md.mustdrop_decode_evict_strided(q, dv["k"], dv["v"], dv["acc"], dv["ids"], dv["protect"], dv["len"], scale, decay,
                                         budget, ev, evc)
        for name in ("k", "v"):
            dv[name] = dv[name].contiguous()
    else:
        md.mustdrop_decode_evict(q, dv["k"], dv["v"], dv["acc"], dv["ids"], dv["protect"], dv["len"], scale, decay, budget,
                                 ev, evc)
    torch.cuda.synchronize()
    g = harness.decode_state_to_host(dv, ev, evc)
    o = {k_: v_.copy() for k_, v_ in s0.items()}
    acc_pre = o["acc"].astype(np.float64)
    r = oracle.decode_evict(t["q_steps"][0], o["k"], o["v"], o["acc"], o["ids"], o["protect"], o["len"], scale, decay, budget)
    o["acc_all"] = (decay * acc_pre + r["a_t"]).astype(np.float32)
    o["evicted_ids"], o["evicted_count"] = r["evicted_ids"], r["evicted_count"]
    check_decode(g, o, s0, budget)
