"""GPU parity of the steady state of a decode loop (one entry leaves, the last one fills its place) around the edges of what the
selection asks for ahead: heads that share the threads unevenly, rows of 1024 vectors and more, entries at the ends of
the rounds, one block per sample and several, and the neighbours of the case (nothing leaves, two leave, protected
entries beyond the budget)."""
import numpy as np
import pytest

import workloads as wl
from parity import check_decode
from test_gpu_decode import gpu_step, initial_state, oracle_step
from test_gpu_decode_shapes import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d,L0,slots", [(4, 64, 65, 66), (4, 128, 1025, 8000), (8, 64, 1024, None), (16, 128, 33, 64), (28, 64, 97, 100),
                                          (32, 64, 1023, 4352), (32, 128, 2049, None), (44, 128, 1024, 2000), (64, 128, 129, None),
                                          (68, 128, 96, None), (128, 64, 1025, 1100)])
@pytest.mark.parametrize("cut", [0, 1, 2])
def test_steady(H, d, L0, slots, cut):
    check(H, d, L0, cut, cut == 1 and H % 8 == 0, slots)


# 60 entries, a budget of 40: one, two or none leave because the others are protected
@pytest.mark.parametrize("H", [12, 32])
@pytest.mark.parametrize("n_protect", [58, 59, 60])
def test_protected_beyond_the_budget(H, n_protect):
    cfg = wl.tiny(wl.CONFIGS[5], B=3, L0=60, steps=1, decode_budget=40, n_protect=n_protect, H=H, d=64)
    t = wl.decode_inputs(cfg, Lcap=200)
    s = initial_state(t)
    g = gpu_step(s, t["q_steps"][0], 0.125, 0.5, 40)
    o = oracle_step(s, t["q_steps"][0], 0.125, 0.5, 40)
    assert np.all(g["len"] == n_protect)
    check_decode(g, o, s, 40)
