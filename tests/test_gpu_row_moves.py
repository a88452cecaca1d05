"""Row moves of the cache cut, bit for bit against hole filling written out: pieces that hold many moves, one, or a part of
one, more pieces than blocks, more than 64 and more than 4096 samples, several layers, samples that move nothing, both cache layouts; and of the
selection where more entries are protected than the budget has room for."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,B,Lcap,H,d", [(1, 70, 40, 4, 64), (3, 2, 300, 40, 128), (2, 1, 64, 8, 512), (2, 2, 50, 128, 128),
                                               (1, 1, 33, 3, 8), (2, 130, 24, 1, 16), (1, 3, 2000, 32, 128), (3, 66, 90, 4, 128),
                                               (2, 2, 700, 65, 64), (2, 1000, 24, 2, 8), (1, 4097, 12, 24, 64), (3, 8300, 10, 1, 8)])
@pytest.mark.parametrize("head_major", [False, True])
def test_hole_filling(layers, B, Lcap, H, d, head_major):
    import torch
    import paper_2411_10803_amd as md
    rng = np.random.default_rng(Lcap * H + B)
    keep = (rng.random((B, Lcap)) < rng.random((B, 1))).astype(np.uint8)
    if B > 2:
        keep[0], keep[1] = 0, 1
    length = rng.integers(Lcap // 2, Lcap + 1, B).astype(np.int32)
    shape = (layers, B, Lcap, H, d)
    kv = [torch.from_numpy(rng.integers(-30000, 30000, shape).astype(np.int16)).cuda() for _ in range(2)]
    want = [x.clone() for x in kv]
    ids = np.stack([rng.permutation(Lcap) for _ in range(B)]).astype(np.int32)
    want_ids, want_len = ids.copy(), length.copy()
    for b in range(B):
        n = int(length[b])
        new = int(keep[b, :n].sum())
        holes = [j for j in range(new) if not keep[b, j]]
        movers = [j for j in range(new, n) if keep[b, j]]
        want_len[b], want_ids[b, holes] = new, ids[b, movers]
        for w in want:
            w[:, b, holes] = w[:, b, movers]
    if head_major:
        kv = [x.transpose(2, 3).contiguous().transpose(2, 3) for x in kv]
    k, v = (x.view(torch.bfloat16) for x in kv)
    t_ids, t_len = torch.from_numpy(ids).cuda(), torch.from_numpy(length).cuda()
    args = (k, v, torch.from_numpy(keep).cuda(), None, t_ids, torch.zeros((B, Lcap), dtype=torch.uint8, device="cuda"), t_len)
    (md.mustdrop_decode_keep_strided if head_major else md.mustdrop_decode_keep)(*args)
    assert (t_len.cpu().numpy() == want_len).all()
    for b in range(B):
        n = int(want_len[b])
        assert (t_ids[b, :n].cpu().numpy() == want_ids[b, :n]).all()
        for got, w in zip((k, v), want):
            assert torch.equal(got.view(torch.int16)[:, b, :n], w[:, b, :n])


@pytest.mark.parametrize("B,Lcap,H,d,budget,protected", [
    (64, 4352, 32, 128, 0, 128), (2, 9000, 32, 128, 5, 500), (1, 1000, 32, 32, 4, 200), (2, 500, 32, 256, 1, 120),
    (1, 9000, 4, 64, 0, 3000), (1, 8200, 3, 128, 5, 5000), (3, 40, 64, 256, 0, 40), (2, 300, 8, 64, 0, 60),
])
@pytest.mark.parametrize("head_major", [False, True])
def test_more_protected_entries_than_budget(B, Lcap, H, d, budget, protected, head_major):
    """Protected entries stay whatever the budget is: the survivors need no scores, K and V must match bit for bit."""
    import torch
    import paper_2411_10803_amd as md
    rng = np.random.default_rng(Lcap + protected)
    g = torch.Generator(device="cuda").manual_seed(Lcap + protected)
    length = rng.integers(protected, Lcap + 1, B).astype(np.int32)
    length[0] = Lcap
    protect = np.zeros((B, Lcap), np.uint8)
    for b in range(B):
        protect[b, rng.choice(int(length[b]), protected, replace=False)] = 1
    # (bf16 patterns of [0, 1))
    kv = [torch.randint(0, 0x3F80, (B, Lcap, H, d), dtype=torch.int16, device="cuda", generator=g) for _ in range(2)]
    want = [x.clone() for x in kv]
    ids = np.stack([rng.permutation(Lcap) for _ in range(B)]).astype(np.int32)
    want_ids = ids.copy()
    for b in range(B):
        keep = protect[b, :length[b]] != 0
        holes = np.flatnonzero(~keep[:protected])
        movers = protected + np.flatnonzero(keep[protected:])
        want_ids[b, holes] = ids[b, movers]
        hd, mv = torch.from_numpy(holes).cuda(), torch.from_numpy(movers).cuda()
        for w in want:
            w[b, hd] = w[b, mv]
    if head_major:
        kv = [x.transpose(1, 2).contiguous().transpose(1, 2) for x in kv]
    k, v = (x.view(torch.bfloat16) for x in kv)
    q = torch.rand((B, H, d), device="cuda", generator=g).to(torch.bfloat16)
    acc = torch.zeros((B, Lcap), device="cuda")
    t_ids, t_len, t_protect = (torch.from_numpy(x).cuda() for x in (ids, length, protect))
    evict = md.mustdrop_decode_evict_strided if head_major else md.mustdrop_decode_evict
    evict(q, k, v, acc, t_ids, t_protect, t_len, d ** -0.5, 1.0, budget)
    assert (t_len.cpu().numpy() == protected).all()
    assert bool((t_protect[:, :protected] == 1).all())
    assert (t_ids.cpu().numpy()[:, :protected] == want_ids[:, :protected]).all()
    for got, w in zip((k, v), want):
        assert torch.equal(got.view(torch.int16)[:, :protected], w[:, :protected])
