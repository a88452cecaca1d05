"""The work whose speed counts in this repository: calls of the three stages through the public entry points.

A case is one call (for a decode step: one append and one evict) as the program around a vision-language model makes
it, on inputs that are already on the GPU, with the output tensors and the workspace it keeps from call to call.

The sizes are the ones of the repository's workloads (24 x 24 patch grids, five tiles, frames of video; 32 heads of
128; prefill budgets of 64 to 512 tokens; a decode cache of 4096 entries cut to 1024) and what lies around and between
them.  The inputs carry the contrast that the method lives on: flat image regions whose neighbouring tokens agree and
textured ones whose tokens do not, a few tokens that the [CLS] token or the prompt attends to and many that it hardly
sees.  Where the decisions fall therefore does not hang on the last bit of a score.
"""
from __future__ import annotations

import math

import torch

import paper_2411_10803_amd as md

TAU = 0.85            # merge threshold: flat windows lie at 0.99, textured ones at 0.5 and below
FLAT_SHARE = 1.0 / 3  # of the image is flat: merging 2x2 windows then leaves three quarters of the tokens
KEY_LAMBDA = 1.0      # the printed key rule, a_cls > mean + lambda * std
BOOST = 4.0           # extra attention logit of a token that matters


def _encode(name, batch, T, H, W, window, dtype, keys, dim=1024, heads=16, adaptive=False):
    kt, kh, kw = window
    return {"name": name, "stage": "encode", "batch": batch, "frames": T, "height": H, "width": W, "kt": kt, "kh": kh,
            "kw": kw, "dtype": dtype, "dim": dim, "heads": heads, "keys": keys, "adaptive": adaptive}


def _prefill(name, batch, vision, text, budget, keys, heads=32, d=128, valid=1.0, lse=False, threshold=False,
             ragged=False, layout="tokens", scores=False):
    return {"name": name, "stage": "prefill", "batch": batch, "vision": vision, "text": text, "budget": budget,
            "keys": keys, "heads": heads, "d": d, "valid": valid, "lse": lse, "threshold": threshold, "ragged": ragged,
            "layout": layout, "scores": scores}


def _step(name, batch, budget, protect, capacity, heads=32, d=128, layout="tokens"):
    return {"name": name, "stage": "step", "batch": batch, "budget": budget, "protect": protect, "capacity": capacity,
            "heads": heads, "d": d, "layout": layout}


def _turn(name, batch, budget, protect, new, heads=32, d=128):
    return {"name": name, "stage": "turn", "batch": batch, "budget": budget, "protect": protect, "new": new,
            "heads": heads, "d": d}


def _keep(name, layers, batch, vision, text, kept, heads=32, d=128):
    return {"name": name, "stage": "keep", "layers": layers, "batch": batch, "vision": vision, "text": text,
            "kept": kept, "heads": heads, "d": d}


def listed():
    return [
        # one image, fp32 features, interactive use: the shortest call, where launches and the host's part count
        _encode("encode_image_f32", 1, 1, 24, 24, (1, 2, 2), "f32", 32),
        # a serving batch of single images
        _encode("encode_images_b16", 16, 1, 24, 24, (1, 2, 2), "bf16", 32),
        # high-resolution images cut into five tiles, the key set by the printed rule
        _encode("encode_tiles_b8", 8, 5, 24, 24, (1, 2, 2), "bf16", 128, adaptive=True),
        # long video clips, merged over space and time
        _encode("encode_video_b2", 2, 16, 24, 24, (2, 2, 2), "bf16", 256),
        # one image and a short question
        _prefill("prefill_image", 1, 576, 32, 192, 32),
        # a serving batch whose attention kernel hands over its row normalisers
        _prefill("prefill_images_lse_b16", 16, 576, 64, 128, 32, valid=0.75, lse=True),
        # high-resolution images after the merge: three quarters of the slots hold tokens
        _prefill("prefill_tiles_b8", 8, 2880, 128, 320, 128, valid=0.75, scores=True),
        # video with prompts of different lengths and a head-major cache, the printed threshold rule
        _prefill("prefill_video_ragged_b3", 3, 4608, 300, 512, 128, valid=0.75, threshold=True, ragged=True,
                 layout="heads"),
        # steady decoding with many sequences: append one entry, evict one
        _step("decode_step_b64", 64, 1024, 128, 4352),
        # the same for a few sequences of a model with 40 heads and a head-major cache
        _step("decode_step_heads40_b4", 4, 777, 64, 1024, heads=40, layout="heads"),
        # a conversation's next turn has filled the cache: cut it back
        _turn("decode_turn_b64", 64, 1024, 128, 3072),
        # hand-over from prefill to decode under the static policy: every layer keeps the same few entries
        _keep("decode_keep_32_layers", 32, 16, 576, 64, 64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; costs at most what the largest listed one does."""
    most = max(work(c)["bytes"] for c in listed())
    while True:
        c = _draw(rng)
        if work(c)["bytes"] <= most:
            del c["name"]
            return c


def _draw(rng):
    stage = rng.choice(("encode", "encode", "encode", "prefill", "prefill", "prefill", "prefill", "step", "step", "turn", "keep"))
    if stage == "encode":
        video = rng.random() < 0.5
        T = rng.randint(2, 16) if video else rng.choice((1, 1, 1, rng.randint(2, 6)))
        H, W = rng.randint(14, 32), rng.randint(14, 32)
        heads = rng.choice((12, 16, 16))
        M = T * H * W
        window = rng.choice(((2, 2, 2), (1, 2, 2))) if video else rng.choice(((1, 2, 2), (1, 2, 2), (1, 3, 3)))
        return _encode("", _log(rng, 1, max(2, 48000 // M)), T, H, W, window, rng.choice(("bf16", "bf16", "bf16", "f32")),
                       max(8, int(M * rng.uniform(0.02, 0.08))), 64 * heads, heads, rng.random() < 0.3)
    if stage == "prefill":
        vision = _log(rng, 128, 9216)
        budget = max(8, int(vision * rng.uniform(0.08, 0.4)))
        return _prefill("", _log(rng, 1, max(2, min(24, 40000 // vision))), vision, _log(rng, 8, 384), budget,
                        int(budget * rng.uniform(0.1, 0.5)), rng.choice((16, 32, 32, 40)), rng.choice((128, 128, 128, 64)),
                        rng.choice((1.0, rng.uniform(0.6, 0.95))), rng.random() < 0.25, rng.random() < 0.3,
                        rng.random() < 0.3, rng.choice(("tokens", "tokens", "heads")), rng.random() < 0.3)
    if stage == "step":
        budget = _log(rng, 128, 4096)
        return _step("", _log(rng, 1, max(2, min(64, 131072 // budget))), budget, budget // rng.randint(4, 16),
                     budget + _log(rng, 16, 3072), rng.choice((16, 32, 32, 40)), rng.choice((128, 128, 128, 64)),
                     rng.choice(("tokens", "heads")))
    if stage == "turn":
        budget = _log(rng, 128, 1024)
        return _turn("", _log(rng, 1, 48), budget, budget // rng.randint(4, 16), int(budget * rng.uniform(2.1, 5)),
                     rng.choice((16, 32, 32, 40)))
    vision = _log(rng, 256, 2880)
    return _keep("", rng.randint(16, 40), _log(rng, 1, 16), vision, _log(rng, 16, 128), int(vision * rng.uniform(0.05, 0.5)),
                 rng.choice((16, 32, 40)))


# ------------------------------------------------------------------------------------------------ inputs

def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, *shape, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(generator=g)


def _random_ranks(g, rows, n):
    """[rows, n]: a random permutation of 0..n-1 in every row."""
    return torch.rand((rows, n), generator=g, device="cuda").argsort(dim=1).argsort(dim=1)


def _lengths(g, batch, n, share):
    """About share * n of n slots per sample, a tenth more or less."""
    if share >= 1.0:
        return torch.full((batch,), n, device="cuda")
    f = share * (0.9 + 0.2 * torch.rand((batch,), generator=g, device="cuda"))
    return (f * n).long().clamp(1, n)


def _by_layout(t, layout):
    """A [.., tokens, heads, d] tensor, or a view of that shape on head-major memory."""
    return t if layout == "tokens" else t.transpose(-3, -2).contiguous().transpose(-3, -2)


def prepare(case, seed):
    made = {"encode": _prepare_encode, "prefill": _prepare_prefill, "step": _prepare_step, "turn": _prepare_turn, "keep": _prepare_keep}
    return made[case["stage"]](case, _generator(seed))


def _prepare_encode(c, g):
    B, T, H, W, D = c["batch"], c["frames"], c["height"], c["width"], c["dim"]
    kt, kh, kw, heads, keys = c["kt"], c["kh"], c["kw"], c["heads"], c["keys"]
    M, dc, dt = T * H * W, D // heads, torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    # regions of 2 x 2 x 2 windows share a content; a region is flat (tokens differ by noise of 0.1) or textured
    rt, rh, rw = -(-T // (2 * kt)), -(-H // (2 * kh)), -(-W // (2 * kw))
    t, y, x = torch.meshgrid(*(torch.arange(n, device="cuda") for n in (T, H, W)), indexing="ij")
    region = ((t // (2 * kt)) * rh * rw + (y // (2 * kh)) * rw + x // (2 * kw)).reshape(-1)
    content = _normal(g, B, rt * rh * rw, D, dtype=torch.float32)
    flat = _random_ranks(g, B, rt * rh * rw) < FLAT_SHARE * rt * rh * rw
    noise = torch.where(flat, 0.1, 1.0)[:, region, None]
    feats = (content[:, region] + noise * _normal(g, B, M, D, dtype=torch.float32)).to(dt)
    q = _normal(g, B, heads, dc, dtype=torch.float32)
    k = _normal(g, B, 1 + M, heads, dc, dtype=torch.float32)
    salient = torch.zeros((B, 1 + M), dtype=torch.bool, device="cuda")
    salient[:, 1:] = _random_ranks(g, B, M) < keys
    k += salient[:, :, None, None] * (BOOST * math.sqrt(dc) * q / q.square().sum(-1, keepdim=True))[:, None]
    i32, u8 = torch.int32, torch.uint8
    new = lambda shape, kind: torch.zeros(shape, dtype=kind, device="cuda")  # noqa: E731
    out = {"out_x": torch.zeros_like(feats), "out_index": new((B, M), i32), "out_mass": new((B, M), torch.float32),
           "out_is_key": new((B, M), u8), "out_valid": new((B, M), u8), "out_count": new((B,), i32),
           "key_index": new((B, keys), i32)}
    if c["adaptive"]:
        out["key_count"] = new((B,), i32)
    return {"stage": "adaptive" if c["adaptive"] else "encode", "x": feats, "q": q.to(dt), "k": k.to(dt),
            "grid": (T, H, W, kt, kh, kw), "keys": keys, "out": out, "result": dict(out),
            "workspace": md.encode_workspace(B, T, H, W, heads, kt, kh, kw)}


def _prepare_prefill(c, g):
    B, Mv, N, R, heads, d, layout = c["batch"], c["vision"], c["text"], c["budget"], c["heads"], c["d"], c["layout"]
    L, C, scale = Mv + N, heads * d, 1.0 / math.sqrt(d)
    mu = math.sqrt(BOOST / math.sqrt(d))
    # after stage 1 a sample's tokens are the first of its slots; some of them are keys, and as many others as the
    # budget has room for are what the prompt asks about
    nv = _lengths(g, B, Mv, c["valid"])
    slot = torch.arange(Mv, device="cuda")[None]
    order = torch.rand((B, Mv), generator=g, device="cuda").masked_fill(slot >= nv[:, None], 2.0).argsort(1).argsort(1)
    valid = (slot < nv[:, None]).to(torch.uint8) if c["valid"] < 1.0 else None
    is_key = ((order < c["keys"]) & (slot < nv[:, None])).to(torch.uint8)
    asked = (order >= c["keys"]) & (order < R) & (slot < nv[:, None])
    q = _normal(g, B, N, heads, d, dtype=torch.float32).add_(mu).bfloat16()
    k = _normal(g, B, L, heads, d)
    k[:, :Mv] += (mu * asked).to(k.dtype)[:, :, None, None]
    txt_len = torch.randint(max(1, N // 3), N + 1, (B,), generator=g, device="cuda").to(torch.int32) if c["ragged"] else None
    rows = Mv if c["threshold"] else R
    i32, u8 = torch.int32, torch.uint8
    new = lambda shape, kind=torch.bfloat16: torch.zeros(shape, dtype=kind, device="cuda")  # noqa: E731
    out = {"hidden_out": new((B, rows + N, C)), "k_out": _by_layout(new((B, rows + N, heads, d)), layout),
           "v_out": _by_layout(new((B, rows + N, heads, d)), layout), "kept_index": new((B, rows), i32),
           "kept_count": new((B,), i32), "out_len": new((B,), i32), "out_protect": new((B, rows + N), u8),
           "out_ids": new((B, rows + N), i32),
           "score_global": new((B, Mv), torch.float32) if c["scores"] else None,
           "score_indiv": new((B, Mv), torch.float32) if c["scores"] else None}
    lse = None
    if c["lse"]:        # what the layer's attention kernel keeps per head and text row
        lse = torch.empty((B, heads, N), dtype=torch.float32, device="cuda")
        causal = torch.ones((N, N), dtype=torch.bool, device="cuda").tril()
        for b in range(B):
            s = torch.matmul(q[b].float().permute(1, 0, 2).contiguous(), k[b].float().permute(1, 2, 0).contiguous()) * scale
            seen = torch.cat([(slot[0] < nv[b])[None].expand(N, Mv), causal], dim=1)
            lse[b] = torch.logsumexp(s.masked_fill(~seen[None], float("-inf")), dim=-1)
    return {"stage": "prefill" if layout == "tokens" else "prefill_heads", "q": _by_layout(q, layout), "k": _by_layout(k, layout),
            "v": _by_layout(_normal(g, B, L, heads, d), layout), "hidden": _normal(g, B, L, C), "valid": valid, "txt_len": txt_len,
            "is_key": is_key, "lse": lse, "Mv": Mv, "scale": scale, "rows": rows, "budget": 0 if c["threshold"] else R,
            "mode": md.FILTER_THRESHOLD if c["threshold"] else md.FILTER_BUDGET, "gamma": 1.0 / Mv, "alpha": (4.0 if c["threshold"] else 2.0) / L,
            "out": out, "result": dict(out), "workspace": md.prefill_workspace(B, Mv, N, heads, rows)}


def _cache_state(g, B, capacity, protect, budget, length):
    ids = torch.arange(capacity, dtype=torch.int32, device="cuda").repeat(B, 1)
    flags = torch.zeros((B, capacity), dtype=torch.uint8, device="cuda")
    flags[:, :budget] = _random_ranks(g, B, budget) < protect
    return {"acc": torch.zeros((B, capacity), dtype=torch.float32, device="cuda"), "ids": ids, "protect": flags,
            "len": torch.full((B,), length, dtype=torch.int32, device="cuda")}


STEPS = 16            # queries and new entries that a decode loop cycles through


def _prepare_step(c, g):
    B, R, cap, heads, d = c["batch"], c["budget"], c["capacity"], c["heads"], c["d"]
    mu = math.sqrt(3.0 / math.sqrt(d))
    k = _normal(g, B, cap, heads, d)
    k += (mu * (torch.rand((B, cap), generator=g, device="cuda") < 0.05)).to(k.dtype)[:, :, None, None]
    k, v = _by_layout(k, c["layout"]), _by_layout(_normal(g, B, cap, heads, d), c["layout"])
    s = _cache_state(g, B, cap, c["protect"], R, R)
    s.update(stage="step" if c["layout"] == "tokens" else "step_heads", k=k, v=v, budget=R, scale=1.0 / math.sqrt(d), count=0, next_id=cap,
             q=(_normal(g, STEPS, B, heads, d) + mu).unbind(0), k_new=_normal(g, STEPS, B, heads, d).unbind(0),
             v_new=_normal(g, STEPS, B, heads, d).unbind(0), evicted=torch.zeros((B, cap), dtype=torch.int32, device="cuda"),
             evicted_count=torch.zeros((B,), dtype=torch.int32, device="cuda"), workspace=md.decode_workspace(B, cap, heads))
    s["result"] = {"k": k[:, :R], "v": v[:, :R], "acc": s["acc"], "ids": s["ids"], "protect": s["protect"], "len": s["len"],
                   "evicted": s["evicted"][:, 0], "evicted_count": s["evicted_count"]}
    return s


def _prepare_turn(c, g):
    B, R, new, heads, d = c["batch"], c["budget"], c["new"], c["heads"], c["d"]
    mu, cap, want = math.sqrt(BOOST / math.sqrt(d)), R + new, R - c["protect"]
    # two turns alternate; each asks about other entries of the new part, as many as the budget has room for
    direction = torch.ones((2, d), device="cuda")
    direction[1, 1::2] = -1.0
    rank = torch.full((B, cap), 3 * want, device="cuda")
    rank[:, R:] = _random_ranks(g, B, new)
    k = _normal(g, B, cap, heads, d)
    for turn in range(2):
        on = (rank // want) == turn
        for b in range(B):
            k[b] += (mu * on[b, :, None, None] * direction[turn]).to(k.dtype)
    v = _normal(g, B, cap, heads, d)
    s = _cache_state(g, B, cap, c["protect"], R, cap)
    q = _normal(g, 2, B, heads, d, dtype=torch.float32) + mu * direction[:, None, None]
    s.update(stage="turn", k=k, v=v, budget=R, scale=1.0 / math.sqrt(d), count=0, full=cap, new=new, q=q.bfloat16().unbind(0),
             new_ids=torch.arange(R, cap, dtype=torch.int32, device="cuda").repeat(B, 1), ids_tail=s["ids"][:, R:],
             acc_tail=s["acc"][:, R:], protect_tail=s["protect"][:, R:],
             evicted=torch.zeros((B, cap), dtype=torch.int32, device="cuda"),
             evicted_count=torch.zeros((B,), dtype=torch.int32, device="cuda"), workspace=md.decode_workspace(B, cap, heads))
    s["result"] = {"k": k[:, :R], "v": v[:, :R], "acc": s["acc"][:, :R], "ids": s["ids"][:, :R], "protect": s["protect"][:, :R],
                   "len": s["len"], "evicted": s["evicted"], "evicted_count": s["evicted_count"]}
    return s


def _prepare_keep(c, g):
    layers, B, Mv, N, kept = c["layers"], c["batch"], c["vision"], c["text"], c["kept"]
    cap, live = Mv + N, kept + N
    k, v = (_normal(g, layers, B, cap, c["heads"], c["d"]) for _ in range(2))
    keep = torch.ones((B, cap), dtype=torch.uint8, device="cuda")
    keep[:, :Mv] = _random_ranks(g, B, Mv) < kept
    ids0 = torch.arange(cap, dtype=torch.int32, device="cuda").repeat(B, 1)
    len0 = torch.full((B,), cap, dtype=torch.int32, device="cuda")
    ids, protect, length = ids0.clone(), keep.clone(), len0.clone()
    return {"stage": "keep", "k": k, "v": v, "keep": keep, "ids0": ids0, "len0": len0, "ids": ids, "protect": protect, "len": length,
            "result": {"k": k[:, :, :live], "v": v[:, :, :live], "ids": ids[:, :live], "protect": protect[:, :live], "len": length},
            "workspace": md.decode_workspace(B, cap, c["heads"])}


# ------------------------------------------------------------------------------------------------ one pass

def run(state):
    s = state
    stage = s["stage"]
    if stage == "encode":
        T, H, W, kt, kh, kw = s["grid"]
        md.mustdrop_encode_merge(s["x"], s["q"], s["k"], None, None, T, H, W, kt, kh, kw, TAU, s["keys"], out=s["out"],
                                 workspace=s["workspace"])
    elif stage == "adaptive":
        T, H, W, kt, kh, kw = s["grid"]
        md.mustdrop_encode_merge_adaptive(s["x"], s["q"], s["k"], None, None, T, H, W, kt, kh, kw, TAU, KEY_LAMBDA, s["keys"],
                                          out=s["out"], workspace=s["workspace"])
    elif stage == "prefill":
        md.mustdrop_prefill_filter(s["q"], s["k"], s["v"], s["hidden"], s["valid"], s["txt_len"], s["is_key"], s["Mv"], s["scale"],
                                   s["mode"], s["budget"], s["gamma"], s["alpha"], Rcap=s["rows"], out=s["out"],
                                   workspace=s["workspace"], row_lse=s["lse"])
    elif stage == "prefill_heads":
        md.mustdrop_prefill_filter_strided(s["q"], s["k"], s["v"], s["hidden"], s["valid"], s["txt_len"], s["is_key"], s["Mv"],
                                           s["scale"], s["mode"], s["budget"], s["gamma"], s["alpha"], s["out"], Rcap=s["rows"],
                                           workspace=s["workspace"], row_lse=s["lse"])
    elif stage in ("step", "step_heads"):
        i, new_id = s["count"] % STEPS, s["next_id"]
        s["count"] += 1
        s["next_id"] += 1
        append, evict = ((md.mustdrop_decode_append, md.mustdrop_decode_evict) if stage == "step" else
                         (md.mustdrop_decode_append_strided, md.mustdrop_decode_evict_strided))
        append(s["k_new"][i], s["v_new"][i], s["k"], s["v"], s["acc"], s["ids"], s["protect"], s["len"], new_id, protect_new=0)
        evict(s["q"][i], s["k"], s["v"], s["acc"], s["ids"], s["protect"], s["len"], s["scale"], 0.0, s["budget"], s["evicted"],
              s["evicted_count"], workspace=s["workspace"])
    elif stage == "turn":
        # the new entries' bookkeeping (their K and V rows are in place), then the cut
        turn = s["count"]
        s["count"] += 1
        torch.add(s["new_ids"], (turn % 4096) * s["new"], out=s["ids_tail"])
        s["acc_tail"].zero_()
        s["protect_tail"].zero_()
        s["len"].fill_(s["full"])
        md.mustdrop_decode_evict(s["q"][turn % 2], s["k"], s["v"], s["acc"], s["ids"], s["protect"], s["len"], s["scale"], 0.0,
                                 s["budget"], s["evicted"], s["evicted_count"], workspace=s["workspace"])
    else:
        s["ids"].copy_(s["ids0"])
        s["protect"].copy_(s["keep"])
        s["len"].copy_(s["len0"])
        md.mustdrop_decode_keep(s["k"], s["v"], s["keep"], None, s["ids"], s["protect"], s["len"], workspace=s["workspace"])
    return s["result"]


# ------------------------------------------------------------------------------------------------ accounting

def work(case):
    """Bytes and operations of one pass: every input row that the method needs once, every output row once."""
    c = case
    if c["stage"] == "encode":
        M, ws = c["frames"] * c["height"] * c["width"], c["kt"] * c["kh"] * c["kw"]
        row = c["dim"] * (4 if c["dtype"] == "f32" else 2)
        left = 1.0 - FLAT_SHARE * (1.0 - 1.0 / ws)
        return {"bytes": c["batch"] * (row * (M + 1 + M + 1 + left * M) + 14.0 * M),
                "flops": c["batch"] * M * c["dim"] * (2.0 + (ws + 1.0))}
    if c["stage"] == "prefill":
        B, N, row = c["batch"], c["text"] * (2.0 / 3 if c["ragged"] else 1.0), c["heads"] * c["d"] * 2.0
        rows = c["valid"] * c["vision"]
        out = c["budget"] + N
        return {"bytes": B * (row * (N + rows + N) + row * (2.0 + 3.0) * out + 16.0 * c["vision"]),
                "flops": 2.0 * B * c["heads"] * c["d"] * N * (rows + N / 2)}
    row = c["heads"] * c["d"] * 2.0
    if c["stage"] == "step":
        live = c["budget"] + 1
        return {"bytes": c["batch"] * (row * (live + 1) + row * (2.0 + 2.0 + 4.0) + 9.0 * live),
                "flops": 2.0 * c["batch"] * live * c["heads"] * c["d"]}
    if c["stage"] == "turn":
        live, moved = c["budget"] + c["new"], c["budget"] - c["protect"]
        return {"bytes": c["batch"] * (row * (live + 1) + row * 3.0 * moved + 17.0 * live),
                "flops": 2.0 * c["batch"] * live * c["heads"] * c["d"]}
    live = c["kept"] + c["text"]
    moved = max(0.0, c["kept"] * (1.0 - live / c["vision"])) + c["text"] if live <= c["vision"] else c["vision"] + c["text"] - live
    return {"bytes": c["layers"] * c["batch"] * row * 4.0 * min(moved, live), "flops": 0.0}


def tolerance(case):
    # measured against float64: merged fp32 rows 4e-8 (largest 1.2e-7), scores 4e-7 (largest 1.4e-6)
    if case["stage"] == "keep" or (case["stage"] == "prefill" and not case["scores"]):
        return "exact"                                 # decisions and copied rows
    if case["stage"] == "encode":
        # merged rows are fp32 means, rounded once to the element type: a bf16 value may land on its neighbour
        return {"rel": 2e-7, "max": 6e-7} if case["dtype"] == "f32" else {"rel": 1e-4, "max": 8e-3}
    return {"rel": 2e-6, "max": 6e-6}                  # sums of fp32 probabilities
