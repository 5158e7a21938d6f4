"""The ping-pong main loop of the prompt-phase GEMMs waits on hand-counted loads, per phase and per tiles that remain:
one and two row tiles of an expert, for every body (64 to 320 rows, full and partly filled), with fewer k-tiles than LDS stages, as many and more, against the oracle."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity

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
