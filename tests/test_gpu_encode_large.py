"""GPU parity of the stage-1 decisions for many tokens per sample: scores made beforehand, tokens in registers and LDS.
Token counts at the edges of the kernel's forms (6144 = 6 x 1024 and so on), windows of 4, 8 and 9 tokens that the
grid clips, both key rules, padding and masses, head counts that are not powers of two."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import check_encode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,win,Hc,extras", [
    (5121, (1, 1, 4), 4, False), (6144, (1, 1, 8), 12, True), (6145, (1, 1, 9), 4, True), (8193, (1, 1, 4), 20, True),
    (10240, (1, 1, 8), 4, False), (12289, (1, 1, 2), 4, True), (16385, (1, 1, 8), 4, False), (28672, (1, 1, 4), 4, True),
    (28673, (1, 1, 4), 4, False)])
def test_many_tokens_per_sample(M, win, Hc, extras):
    from paper_2411_10803_amd import harness
    kt, kh, kw = win
    B, dc = 2, 8
    rng = np.random.default_rng(M)
    D = Hc * dc
    x = np.repeat(rng.standard_normal((B, -(-M // kw), D), dtype=np.float32), kw, axis=1)[:, :M]
    x = x + np.float32(rng.choice([0.05, 1.0], size=(B, -(-M // kw), 1)).repeat(kw, axis=1)[:, :M]) * rng.standard_normal((B, M, D), dtype=np.float32)
    x = wl.f32_to_bf16_bits(x)
    q = wl.f32_to_bf16_bits(rng.standard_normal((B, Hc, dc), dtype=np.float32))
    k = wl.f32_to_bf16_bits(rng.standard_normal((B, 1 + M, Hc, dc), dtype=np.float32))
    valid = (rng.random((B, M)) > 0.1).astype(np.uint8) if extras else None
    mass = rng.integers(1, 5, size=(B, M)).astype(np.float32) if extras else None
    args = (1, 1, M, kt, kh, kw, 0.7)
    print(f"M={M} window={win} Hc={Hc} extras={extras}", flush=True)
    g = harness.encode_on_gpu(x, wl.BF16, q, k, wl.BF16, mass, valid, *args, 100)
    o = oracle.encode_merge(x, wl.BF16, q, k, wl.BF16, mass, valid, *args, 100)
    s = check_encode(g, o, x, wl.BF16, valid, *args, 100)
    assert s["merged_rows_checked"] > 50 and s["copied_rows_checked"] > 1000
    g = harness.encode_on_gpu(x, wl.BF16, None, None, wl.BF16, mass, valid, *args, 0)           # no key set at all
    o = oracle.encode_merge(x, wl.BF16, None, None, wl.BF16, mass, valid, *args, 0)
    check_encode(g, o, x, wl.BF16, valid, *args, 0)
    args = args[:7] + (2.0, 64)                                                                 # Eq. 7 as printed
    g = harness.encode_adaptive_on_gpu(x, wl.BF16, q, k, wl.BF16, mass, valid, *args)
    o = oracle.encode_merge_adaptive(x, wl.BF16, q, k, wl.BF16, mass, valid, *args)
    check_encode(g, o, x, wl.BF16, valid, *args[:7], 64, key_lambda=2.0)


# more heads than the decision kernel merges itself: the general kernel for few tokens, ready-made scores for more
@pytest.mark.parametrize("B,M,Hc", [(3, 7, 20), (3, 384, 64), (3, 385, 64), (1, 768, 64), (1, 769, 64), (2, 1024, 24), (2, 1025, 24)])
def test_more_than_sixteen_heads(B, M, Hc):
    from paper_2411_10803_amd import harness
    rng = np.random.default_rng(M)
    x = wl.f32_to_bf16_bits(rng.standard_normal((B, M, Hc * 8), dtype=np.float32))
    q = wl.f32_to_bf16_bits(rng.standard_normal((B, Hc, 8), dtype=np.float32))
    k = wl.f32_to_bf16_bits(rng.standard_normal((B, 1 + M, Hc, 8), dtype=np.float32))
    valid = (rng.random((B, M)) > 0.2).astype(np.uint8)
    args = (1, 1, M, 1, 1, 4, 0.0, 3)
    g = harness.encode_on_gpu(x, wl.BF16, q, k, wl.BF16, None, valid, *args)
    o = oracle.encode_merge(x, wl.BF16, q, k, wl.BF16, None, valid, *args)
    check_encode(g, o, x, wl.BF16, valid, *args)
