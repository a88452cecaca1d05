"""The row statistics where a wave holds all text blocks of a group, against torch's normalisers in 64 bits: the scores of a
call that computes its own must be those of a call that is handed torch's."""
import pytest

pytestmark = pytest.mark.gpu


def normalisers(torch, q, k, Mv, valid, txt_len, scale):
    B, N, H, _ = q.shape
    lse = torch.zeros((B, H, N), dtype=torch.float32, device="cuda")
    causal = torch.ones((N, N), dtype=torch.bool, device="cuda").tril()
    for b in range(B):
        vis = valid[b].bool() if valid is not None else torch.ones(Mv, dtype=torch.bool, device="cuda")
        seen = torch.cat([vis[None].expand(N, Mv), causal], 1)
        for h in range(H):
            s = torch.mm(q[b, :, h].double(), k[b, :, h].double().t().contiguous()) * scale
            lse[b, h] = torch.logsumexp(s.masked_fill(~seen, float("-inf")), -1)
    return lse


def compare(torch, q, k, v, hidden, Mv, valid, txt, scale):
    import paper_2411_10803_amd as md
    N = q.shape[1]
    txt_len = torch.tensor(txt, dtype=torch.int32, device="cuda") if txt else None
    lse = normalisers(torch, q, k, Mv, valid, txt_len, scale)
    got = []
    for given in (None, lse):
        out = md.mustdrop_prefill_filter(q, k, v, hidden, valid, txt_len, None, Mv, scale, md.FILTER_BUDGET, 1, 1.0 / Mv,
                                         2.0 / (Mv + N), 1, row_lse=given)
        got.append((out["score_global"].double(), out["score_indiv"].double()))
    # a normaliser is a sum of at most 270 tiles per lane and a few merges of fp32 terms: 300 * 2^-24
    for own, handed in zip(*got):
        assert bool(torch.isfinite(own).all())
        assert bool(((own - handed).abs() <= 2e-5 * handed.abs()).all()), float((own - handed).abs().max())


@pytest.mark.parametrize("B,Mv,N,H,d,mask,txt", [
    (1, 1, 129, 1, 128, None, None),                     # text keys only, but for one
    (2, 31, 160, 2, 128, "holes", [160, 129]),           # groups of three and two; mask rows off a word
    (2, 33, 193, 3, 64, "prefix", [193, 5]),             # four and three; groups without rows
    (2, 127, 257, 2, 128, "none", [257, 0]),             # three groups of three; no valid slot
    (3, 2048, 300, 4, 128, "prefix", [300, 200, 97]),    # one word of the mask row per lane
    (2, 2052, 130, 4, 64, "holes", None),                # and a second one
    (1, 10302, 140, 2, 128, "holes", None),              # more slots than the one look at the mask row covers
    (2, 8448, 129, 128, 64, "holes", [129, 129]),        # more than 64 tiles per wave
    (16, 600, 70, 32, 128, "prefix", None),              # one text group, blocks of four waves
    (17, 290, 128, 31, 128, "holes", None),
])
def test_row_statistics(B, Mv, N, H, d, mask, txt):
    import torch
    g = torch.Generator(device="cuda").manual_seed(B * Mv + N)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)  # noqa: E731
    q, k = normal(B, N, H, d), normal(B, Mv + N, H, d)
    v, hidden, scale = k, normal(B, Mv + N, 8), d ** -0.5
    valid = None
    if mask:
        share = torch.rand((B, 1), generator=g, device="cuda")
        slot = torch.arange(Mv, device="cuda")[None] / Mv
        valid = {"prefix": slot <= share, "none": slot < -share,
                 "holes": (torch.rand((B, Mv), generator=g, device="cuda") < 0.9) & (slot <= 0.5 + 0.5 * share)}[mask].to(torch.uint8).contiguous()
    compare(torch, q, k, v, hidden, Mv, valid, txt, scale)


@pytest.mark.parametrize("N,d,counts", [(160, 128, [0, 1, 40]), (160, 64, [0, 1, 40]), (300, 128, [33, 0, 300])])
def test_waves_without_tiles(N, d, counts):
    """Seven or eight key chunks, of which the valid slots leave one to three: waves and whole blocks go without a tile."""
    import torch
    B, Mv, H = len(counts), 4096, 8
    g = torch.Generator(device="cuda").manual_seed(N + d)
    normal = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)  # noqa: E731
    q, k, hidden = normal(B, N, H, d), normal(B, Mv + N, H, d), normal(B, Mv + N, 8)
    valid = (torch.arange(Mv, device="cuda")[None] < torch.tensor(counts, device="cuda")[:, None]).to(torch.uint8).contiguous()
    compare(torch, q, k, k, hidden, Mv, valid, None, d ** -0.5)
