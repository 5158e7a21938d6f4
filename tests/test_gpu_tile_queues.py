"""The tile queues of the prompt-phase GEMMs against the oracle: every body (32 to 320 rows in steps of 32, and one row on
either side), launches of less than a round to several, last rounds that are cut along columns and along rows, spill tiles and
short last tiles, experts without rows, and a second call on the same layer (the counters start over)."""
import numpy as np
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_ff", [320, 8256])
def test_every_body(oracle, d_ff):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=192, d_ff=d_ff, seed=900 + d_ff)
    w = synth.make_weights(cfg)
    xp = synth.make_tokens(cfg, 600)
    yo = oracle.layer_forward(xp, w["w_gate"], w["w_up"], w["w_down"])
    L = GpuLayer(cfg, w, (1.0, 0.0, 0.0), max_tokens=600)
    try:
        for T in [b + d for b in range(32, 321, 32) for d in (-1, 0, 1)] + [512, 560, 576, 600]:
            print("body H=%d T=%d" % (d_ff, T), flush=True)
            assert_parity(L.forward(xp[:T], None, mode=si.SI_PREFILL), yo[:T])
    finally:
        L.close()


# gate/up tiles of 128 columns: one row tile x 300 (1.2 rounds of 256, cut along columns up to 160 rows, above along rows),
# then several row tiles; n_g: the CG' launches, which take the X2 rows only
@pytest.mark.parametrize("T,d_ff,split,n_g", [(150, 38400, (1.0, 0.0, 0.0), 0), (200, 38400, (1.0, 0.0, 0.0), 0), (300, 38400, (1.0, 0.0, 0.0), 0),
                                              (513, 17408, (1.0, 0.0, 0.0), 0), (577, 8704, (0.5, 0.0, 0.5), 320), (90, 8704, (0.5, 0.25, 0.25), 90)])
def test_cut_tiles_dense(oracle, T, d_ff, split, n_g):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=64, d_ff=d_ff, seed=31)
    w = synth.make_weights(cfg)
    xp = synth.make_tokens(cfg, T)
    yo = oracle.layer_forward(xp, w["w_gate"], w["w_up"], w["w_down"])
    L = GpuLayer(cfg, w, split, max_tokens=T)
    try:
        for _ in range(2):
            assert_parity(L.forward(xp, None, mode=si.SI_PREFILL, n_g=n_g), yo)
    finally:
        L.close()


@pytest.mark.parametrize("E,k,T,d_ff,d_ff_shared,n_g", [(6, 1, 900, 1280, 0, 0), (16, 2, 300, 2560, 0, 0), (5, 2, 700, 704, 1344, 0), (6, 2, 640, 512, 0, 600), (64, 8, 96, 256, 320, 0)])
def test_experts_of_unequal_rows(oracle, E, k, T, d_ff, d_ff_shared, n_g):
    split = (1.0, 0.0, 0.0) if n_g == 0 else (0.5, 0.25, 0.25)
    cfg = synth.scaled(synth.CONFIGS["qwen_moe"], d_model=128, d_ff=d_ff, d_ff_shared=d_ff_shared, n_experts=E, top_k=k, seed=70 + E)
    w = synth.make_weights(cfg)
    xp = synth.make_tokens(cfg, T)
    lg = np.random.default_rng(E).standard_normal((T, E)).astype(np.float32)
    lg[:, 0] += 2.0            # one expert with most rows, the last without any
    lg[:, E - 1] -= 100.0
    lg[::3, 1] += 4.0
    shared = (w["s_gate"], w["s_up"], w["s_down"]) if d_ff_shared else None
    yo = oracle.layer_forward(xp, w["w_gate"], w["w_up"], w["w_down"], logits=lg, top_k=k, shared=shared)
    L = GpuLayer(cfg, w, split, max_tokens=T)
    try:
        for n in (n_g, n_g, 0):
            print("unequal E=%d T=%d n_g=%d" % (E, T, n), flush=True)
            assert_parity(L.forward(xp, lg, mode=si.SI_PREFILL, n_g=n), yo)
    finally:
        L.close()


@pytest.mark.parametrize("d_model,d_ff", [(64, 320), (192, 768), (576, 1024), (1024, 2112)])
def test_every_body_q4(oracle, d_model, d_ff):
    """4-bit bodies, with 1 to 16 k-tiles (odd numbers of scale groups per row among them); codes and scales as in earnest."""
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff, seed=40 + d_model)
    wq = synth.make_weights_q4(cfg)
    for key in ("z_gate", "z_up", "z_down"):
        wq[key] = (wq[key] & 0xFF80) | 0x20  # scales of three significant bits: a weight has at most 7 and is a bfloat16
    xp = synth.make_tokens(cfg, 600)
    yo = oracle.layer_forward_q4(xp, wq)
    L = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=600)
    try:
        for T in [b + d for b in range(32, 257, 32) for d in (-1, 0, 1)] + [300, 320, 560, 576, 600]:
            print("4-bit body M=%d H=%d T=%d" % (d_model, d_ff, T), flush=True)
            assert_parity(L.forward(xp[:T], None, mode=si.SI_PREFILL), yo[:T])
    finally:
        L.close()
