"""GPU parity of the survivors' rows where the deciding blocks write them and around the line where a launch of its own does:
token counts at the edges of the decision kernel's forms, clipped windows, rows that are no whole number of 64-vector
slices, samples with more and with fewer blocks than the small outputs have waves, masses and padding."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import check_encode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,M,win,D,bf16,extras", [
    (1, 1, (1, 1, 2), 8, True, False), (1, 3, (1, 1, 4), 16, False, True), (2, 1023, (1, 1, 4), 72, True, True),
    (3, 1025, (1, 1, 8), 520, True, True), (1, 2049, (1, 1, 5), 264, False, True), (2, 3072, (1, 1, 4), 48, True, False),
    (1, 3073, (1, 1, 7), 40, True, True), (1, 5120, (1, 1, 4), 80, False, True), (1, 5120, (1, 1, 8), 64, True, False),
    (17, 130, (1, 1, 4), 1032, True, True), (128, 37, (1, 1, 2), 32, True, True), (129, 37, (1, 1, 2), 32, True, True),
    (2, 90, (1, 1, 9), 136, True, True), (86, 129, (1, 1, 4), 32, True, True), (102, 256, (1, 1, 2), 16, False, False), (103, 256, (1, 1, 4), 32, True, True)])
def test_rows(B, M, win, D, bf16, extras):
    from paper_2411_10803_amd import harness
    kt, kh, kw = win
    dt = wl.BF16 if bf16 else wl.F32
    rng = np.random.default_rng(M * D)
    x = np.repeat(rng.standard_normal((B, -(-M // kw), D), dtype=np.float32), kw, axis=1)[:, :M]
    x = x + np.float32(rng.choice([0.05, 1.0], size=(B, -(-M // kw), 1)).repeat(kw, axis=1)[:, :M]) * rng.standard_normal((B, M, D), dtype=np.float32)
    x = wl.f32_to_bf16_bits(x) if bf16 else x
    valid = (rng.random((B, M)) > 0.1).astype(np.uint8) if extras else None
    mass = rng.integers(1, 5, size=(B, M)).astype(np.float32) if extras else None
    keys, dc = min(M, 5), 8                              # heads of eight features, as many as fit; fewer for wide rows
    q = k = None
    Hc = D // dc
    if Hc <= 16:
        q = rng.standard_normal((B, Hc, dc), dtype=np.float32)
        k = rng.standard_normal((B, 1 + M, Hc, dc), dtype=np.float32)
    else:
        keys = 0
    args = (1, 1, M, kt, kh, kw, 0.7, keys)
    print(f"B={B} M={M} window={win} D={D} bf16={bf16} extras={extras} keys={keys}", flush=True)
    g = harness.encode_on_gpu(x, dt, q, k, wl.F32, mass, valid, *args)
    o = oracle.encode_merge(x, dt, q, k, wl.F32, mass, valid, *args)
    check_encode(g, o, x, dt, valid, *args)


def test_rows_with_outputs_over_inputs():
    """Masses that are written over the ones read (nothing merges, so that a launch of its own gives the rows)."""
    import torch
    import paper_2411_10803_amd as md
    B, M, D = 2, 700, 64
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.standard_normal((B, M, D), dtype=np.float32)).cuda()
    mass = torch.from_numpy(rng.integers(1, 5, size=(B, M)).astype(np.float32)).cuda()
    want = mass.clone()
    out = md.mustdrop_encode_merge(x, None, None, mass, None, 1, 1, M, 1, 1, 2, 2.0, 0)
    got = md.mustdrop_encode_merge(x, None, None, mass, None, 1, 1, M, 1, 1, 2, 2.0, 0, out=dict(out, out_mass=mass))
    assert torch.equal(got["out_mass"], want) and torch.equal(got["out_x"], x) and torch.equal(out["out_x"], x)


@pytest.mark.parametrize("name", ["out_mass", "out_index", "out_is_key", "out_valid", "out_count", "key_index", "key_count", "a_cls", "window_sim"])
def test_every_output_over_the_masses(name):
    """The same for each output, with tokens missing, so that what is written differs from what was there: the decisions are one
    block's, and the rows have a launch of their own."""
    import torch
    import paper_2411_10803_amd as md
    from paper_2411_10803_amd import binding
    M, D, keys = 700, 64, 40
    rng = np.random.default_rng(6)
    dev = lambda a: torch.from_numpy(a).cuda()                                                       # noqa: E731
    x, q, k = (dev(rng.standard_normal(s, dtype=np.float32)) for s in ((1, M, D), (1, 4, 16), (1, 1 + M, 4, 16)))
    valid = dev((rng.random((1, M)) > 0.3).astype(np.uint8))
    mass = dev(rng.integers(1, 5, size=(1, M)).astype(np.float32))
    call = lambda m, out=None: md.mustdrop_encode_merge_adaptive(x, q, k, m, valid, 1, 1, M, 1, 1, 2, 2.0, 1.0, keys, out=out)  # noqa: E731
    want = {n: t.clone() for n, t in call(mass.clone()).items() if n != "workspace"}
    n = int(want["out_count"][0])
    assert n < 600
    fresh = {n_: torch.zeros_like(t) for n_, t in want.items()}
    fresh[name] = mass.view(-1).view(want[name].dtype)[:want[name].numel()].view(want[name].shape)
    binding.profile_start()
    got = call(mass, fresh)
    torch.cuda.synchronize()
    assert "encode_emit" in binding.profile_stop()
    for n_, t in want.items():
        rows = n if n_ in ("out_x", "out_index", "out_mass", "out_is_key") else t.shape[1] if t.dim() > 1 else 1
        assert torch.equal(got[n_][:, :rows] if t.dim() > 1 else got[n_], t[:, :rows] if t.dim() > 1 else t), n_


def test_rows_beyond_the_cache():
    """240 MB of features in one call, whose rows have a launch of their own, and in two, whose deciding blocks write them."""
    import torch
    import paper_2411_10803_amd as md
    from paper_2411_10803_amd import binding
    B, M, D, Hc, keys = 102, 576, 1024, 16, 32
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty((B, M // 4, 1, D), device="cuda").normal_(generator=g).expand(B, M // 4, 4, D).reshape(B, M, D).clone()
    x += torch.empty((B, M, D), device="cuda").normal_(generator=g) * (torch.rand((B, M // 4, 1, 1), generator=g, device="cuda") > 0.4).float().expand(
        B, M // 4, 4, 1).reshape(B, M, 1)
    q = torch.empty((B, Hc, D // Hc), device="cuda").normal_(generator=g)
    k = torch.empty((B, 1 + M, Hc, D // Hc), device="cuda").normal_(generator=g)
    call = lambda a, b: md.mustdrop_encode_merge(x[a:b], q[a:b], k[a:b], None, None, 1, 1, M, 1, 1, 4, 0.85, keys)  # noqa: E731
    launched, outs = [], []
    for a, b in ((0, B), (0, B // 2), (B // 2, B)):
        binding.profile_start()
        outs.append(call(a, b))
        torch.cuda.synchronize()
        launched.append(sorted(binding.profile_stop()))
    assert "encode_emit" in launched[0] and "encode_decide_emit" in launched[1] and "encode_decide_emit" in launched[2]
    assert int(outs[0]["out_count"].max()) < M
    for n in ("out_x", "out_index", "out_mass", "out_is_key", "out_valid", "out_count", "key_index", "a_cls", "window_sim"):
        assert torch.equal(outs[0][n], torch.cat([outs[1][n], outs[2][n]])), n
