"""The 4-bit generation-phase kernels at the edges of their splits, against the oracle: d_model of half a load unit, of
odd scale-group counts and of fewer units than waves; slots of one, two, odd and many chunks; 1 to 16 tokens (one pass
over the weights or several, operand rows partly filled).  Products are exact and sums fp32, so the result is held to
1e-4 x RMS (measured 1e-5: the sums cancel a 136-fold offset) instead of the bf16 tolerance."""
import numpy as np
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,d_ff", [(64, 64), (128, 192), (192, 576), (320, 1088), (576, 4096), (1024, 2048), (8192, 640)])
def test_q4_gemv_edges(oracle, d_model, d_ff):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff, seed=700 + d_model)
    wq = synth.make_weights_q4(cfg)
    L = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=16)
    try:
        xp = synth.make_tokens(cfg, 16)
        yo = oracle.layer_forward_q4(xp, wq)
        for T in (1, 2, 3, 4, 5, 8, 9, 16):
            print("4-bit GEMV M=%d H=%d T=%d" % (d_model, d_ff, T), flush=True)
            assert_parity(L.forward(xp[:T], None, mode=si.SI_DECODE), yo[:T], tol=1e-4)
    finally:
        L.close()


@pytest.mark.parametrize("d_model,d_ff", [(576, 192), (512, 1024), (4096, 3584)])
def test_q4_down_projection_outliers(oracle, d_model, d_ff):
    """FC2 alone: the activations h = 64 u are exact in fp32 (gate 64, whose SiLU is 64; u a sum of three codes times powers of
    two), 1 % of them 512 times the others, with codes at 8 (weight 0) or next to it, and rows scaled down to 2^-100.  h * w
    is exact in fp32 and every sum is one, so a result may be off by a rounding of at most 2^-24 of sum |h w| for each of the
    64 terms of a group, its parts and scale, the up to 16 groups of a slot and the up to 16 slots: 100 * 2^-24 * sum |h w|
    (measured: 1.3; sums that carry an offset of 136 until it cancels: 490; 8: 112)."""
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff)
    rng = np.random.default_rng(d_model + d_ff)
    bf16 = lambda a: (np.ascontiguousarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16)  # (of values that are bf16)
    pack = lambda q: (q[..., 0::2] | (q[..., 1::2] << 4)).astype(np.uint8)[None]
    draw = lambda shape: np.clip(np.round(rng.standard_normal(shape) * 2.4) + 8, 0, 15).astype(np.uint8)
    gate, up, down = np.full((d_ff, d_model), 8, np.uint8), np.full((d_ff, d_model), 8, np.uint8), draw((d_ff, d_model))
    gate[:, 0] = 9
    up[:, 64:67] = draw((d_ff, 3))
    z_up = np.full((d_ff, d_model // 64), 2.0 ** -6)
    big = rng.choice(d_ff, max(1, d_ff // 100), replace=False)
    z_up[big] = 8.0
    down[big] = 8 + rng.integers(-1, 2, (len(big), d_model)) * (rng.random((len(big), d_model)) < 0.1)
    z_down = (rng.integers(128, 256, (d_ff // 64, d_model)) * 2.0 ** -14).astype(np.float32)
    wq = {"q_gate": pack(gate), "q_up": pack(up), "q_down": pack(down), "z_gate": bf16(np.full((d_ff, d_model // 64), 64.0))[None],
          "z_up": bf16(z_up)[None], "z_down": bf16(z_down)[None]}
    T = 5
    x = np.zeros((T, d_model), np.float32)
    x[:, 0] = 1.0
    x[:, 64:67] = np.array([1.0, 2.0 ** -6, 2.0 ** -12]) * np.array([1.0, -2.0, 2.0 ** -40, 2.0 ** 20, 2.0 ** -100])[:, None]
    xb = bf16(x)
    yo = oracle.layer_forward_q4(xb, wq)
    u = (x[:, 64:67].astype(np.float64) @ (up[:, 64:67].astype(np.float64) - 8).T) * z_up[:, 1]
    bound = 100 * 2.0 ** -24 * (np.abs(64 * u) @ (np.abs(down.astype(np.float64) - 8) * np.repeat(z_down.astype(np.float64), 64, axis=0)))
    L = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=8)
    try:
        for n in (1, T):
            print("4-bit down projection, outliers M=%d H=%d T=%d" % (d_model, d_ff, n), flush=True)
            y = L.forward(xb[:n], None, mode=si.SI_DECODE).astype(np.float64)
            assert np.all(np.abs(y - yo[:n]) <= bound[:n]), float(np.max(np.abs(y - yo[:n]) / np.maximum(bound[:n], 1e-300)))
    finally:
        L.close()
