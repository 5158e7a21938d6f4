"""The bf16 generation-phase kernels at the edges of their splits, against the oracle: rows of x of less than a wave, of
several staging batches and of a remainder; j-slots of one chunk (small layers) to many; 1 to 9 tokens (one pass over the
weights or several, the last one partly filled); one expert and several.  Exact products, fp32 sums: 1e-4 x RMS."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k", [(1, 1), (4, 2)])
@pytest.mark.parametrize("d_model,d_ff", [(64, 64), (192, 1088), (576, 2112), (1088, 320), (3328, 2240), (8192, 192)])
def test_decode_edges(oracle, d_model, d_ff, E, k):
    base = synth.CONFIGS["llama2_70b" if E == 1 else "mixtral_8x7b"]
    cfg = synth.scaled(base, d_model=d_model, d_ff=d_ff, n_experts=E, top_k=k, seed=900 + d_model)
    w = synth.make_weights(cfg)
    L = GpuLayer(cfg, w, (1.0, 0.0, 0.0), max_tokens=16)
    try:
        for T in (1, 2, 3, 4, 5, 9):
            print("decode M=%d H=%d E=%d T=%d" % (d_model, d_ff, E, T), flush=True)
            xb = synth.make_tokens(cfg, T)
            lg = synth.make_router_logits(cfg, xb)
            yo = oracle.layer_forward(xb, w["w_gate"], w["w_up"], w["w_down"], logits=lg, top_k=k)
            assert_parity(L.forward(xb, lg, mode=si.SI_DECODE), yo, tol=1e-4)
    finally:
        L.close()
