"""The 4-bit generation-phase kernels at the edges of their splits, against the oracle: d_model of half a load unit, of
odd scale-group counts and of fewer units than waves; slots of one, two, odd and many chunks; 1 to 16 tokens (one pass
over the weights or several, operand rows partly filled).  Products are exact and sums fp32, so the result is held to
1e-4 x RMS (measured 1e-5: the sums cancel a 136-fold offset) instead of the bf16 tolerance."""
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
