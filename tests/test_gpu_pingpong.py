"""The ping-pong main loop of the prompt-phase GEMMs waits on hand-counted loads, per phase and per tiles that remain:
one and two row tiles of an expert, for every body (64 to 320 rows, full and partly filled), with fewer k-tiles than LDS stages, as many and more, against the oracle."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu

# one tile on both sides of each body, then 256 + 65, 256 + 128, 256 + 129, 256 + 192, 256 + 256, 256 + 257, 256 + 320
ROWS = (64, 65, 128, 129, 192, 193, 321, 384, 385, 448, 512, 513, 576)


@pytest.mark.parametrize("d_model,d_ff", [(64, 64), (128, 512), (192, 768), (256, 1088), (320, 1600), (448, 2048)])
def test_pingpong_bodies(oracle, d_model, d_ff):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff, seed=500 + d_model)
    w = synth.make_weights(cfg)
    L = GpuLayer(cfg, w, (1.0, 0.0, 0.0), max_tokens=max(ROWS))
    try:
        xp = synth.make_tokens(cfg, max(ROWS))
        yo = oracle.layer_forward(xp, w["w_gate"], w["w_up"], w["w_down"])
        for T in ROWS:
            print("ping-pong M=%d H=%d T=%d" % (d_model, d_ff, T), flush=True)
            assert_parity(L.forward(xp[:T], None, mode=si.SI_PREFILL), yo[:T])
    finally:
        L.close()


@pytest.mark.parametrize("d_model,d_ff", [(64, 64), (192, 704), (448, 1024)])
def test_one_barrier_bodies(oracle, d_model, d_ff):
    """The bodies with one barrier per k-tile (64 rows bf16, 64 and 128 rows 4-bit) and their neighbours, few rows too."""
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff, seed=600 + d_model)
    w, wq = synth.make_weights(cfg), synth.make_weights_q4(cfg)
    xp = synth.make_tokens(cfg, 385)
    yo, yq = oracle.layer_forward(xp, w["w_gate"], w["w_up"], w["w_down"]), oracle.layer_forward_q4(xp, wq)
    L, Q = GpuLayer(cfg, w, (1.0, 0.0, 0.0), max_tokens=385), Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=385)
    try:
        for T in (1, 17, 33, 64, 65, 128, 129, 192, 193, 257, 320, 385):
            print("one barrier M=%d H=%d T=%d" % (d_model, d_ff, T), flush=True)
            assert_parity(L.forward(xp[:T], None, mode=si.SI_PREFILL), yo[:T])
            # the path's own roundings (weights and activations to bf16), applied in double, reach 2.14e-2 x RMS on the
            # 64 x 64 layer (64 terms per sum average little) and 1.5e-2 on the others
            assert_parity(Q.forward(xp[:T], None, mode=si.SI_PREFILL), yq[:T], tol=2.5e-2)
    finally:
        L.close()
        Q.close()
