"""GPU parity of the score pass where key rows are cut into slices of the feature dimension (a last slice that is not
full, heads of several widths, padding) and of windows of nine members next to the forms around them."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity import check_encode
from test_gpu_encode import both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,Hg,Wg,win,Hc,dc,bf16", [
    (1, 13, 17, (1, 3, 3), 12, 64, True), (1, 13, 17, (1, 3, 3), 12, 64, False), (1, 24, 24, (1, 2, 2), 9, 64, True),
    (2, 9, 9, (1, 3, 3), 5, 128, False), (1, 11, 8, (2, 2, 2), 16, 32, True), (1, 8, 30, (1, 2, 5), 20, 64, False),
    (1, 6, 6, (1, 3, 3), 3, 512, True)])
def test_slices(T, Hg, Wg, win, Hc, dc, bf16):
    dt = wl.BF16 if bf16 else wl.F32
    kt, kh, kw = win
    cfg = wl.tiny(wl.CONFIGS[2], B=3, T=T, Hg=Hg, Wg=Wg, D=Hc * dc, Hc=Hc, dc=dc, kt=kt, kh=kh, kw=kw, x_dtype=dt, key_budget=7)
    e = wl.encode_inputs(cfg)
    rng = np.random.default_rng(Hc * dc)
    valid = (rng.random((cfg.B, cfg.M)) > 0.2).astype(np.uint8)
    o0 = oracle.encode_merge(e["x"], dt, None, None, dt, None, valid, T, Hg, Wg, kt, kh, kw, 2.0, 0)
    tau = float(np.median(o0["window_sim"]))
    g, o = both(e["x"], dt, e["q_cls"], e["k_cls"], dt, None, valid, T, Hg, Wg, kt, kh, kw, tau, 7)
    check_encode(g, o, e["x"], dt, valid, T, Hg, Wg, kt, kh, kw, tau, 7)
