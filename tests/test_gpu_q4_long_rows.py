"""4-bit generation calls over several experts with the longest rows, against the oracle: from four tokens on, x of d_model 8192 is staged in
LDS without padding, its pieces in an order of each token's own (8128 is the last d_model with padding).  Products are exact and sums fp32: 1e-4 x RMS."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model", [8128, 8192])
@pytest.mark.parametrize("d_ff,d_ff_shared", [(64, 0), (128, 0), (64, 192), (192, 64)])
def test_long_rows(oracle, d_model, d_ff, d_ff_shared):
    cfg = synth.scaled(synth.CONFIGS["qwen_moe"], d_model=d_model, d_ff=d_ff, d_ff_shared=d_ff_shared, n_experts=4, top_k=2, seed=d_model + d_ff)
    wq = synth.make_weights_q4(cfg)
    L = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=16)
    try:
        for T in (3, 4, 5, 9, 16):
            print("long rows M=%d H=%d+%d T=%d" % (d_model, d_ff, d_ff_shared, T), flush=True)
            xp = synth.make_tokens(cfg, T, stream=T)
            lg = synth.make_router_logits(cfg, xp)
            assert_parity(L.forward(xp, lg, mode=si.SI_DECODE), oracle.layer_forward_q4(xp, wq, logits=lg, top_k=cfg.top_k), tol=1e-4)
    finally:
        L.close()
