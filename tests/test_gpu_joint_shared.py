"""Routed and shared experts in one launch, against the oracle: shared experts narrower than, as wide as and many times as
wide as a routed one (part of the last grid row empty, several grid rows), one and several routed experts, the token
assignment inside the launch (up to 8 pairs) and before it, and slicing rates that leave either kind resident or not."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q4", [False, True])
@pytest.mark.parametrize("E,k,d_ff,d_ff_shared,split", [
    (1, 1, 192, 320, (1.0, 0.0, 0.0)), (1, 1, 320, 192, (0.4, 0.3, 0.3)), (4, 2, 192, 64, (1.0, 0.0, 0.0)), (4, 2, 192, 192, (1.0, 0.0, 0.0)), (12, 3, 128, 1088, (1.0, 0.0, 0.0)),
    (2, 1, 64, 4160, (1.0, 0.0, 0.0)), (4, 1, 576, 320, (0.5, 0.5, 0.0)), (4, 2, 64, 320, (0.3, 0.4, 0.3))])
def test_joint(oracle, q4, E, k, d_ff, d_ff_shared, split):
    cfg = synth.scaled(synth.CONFIGS["qwen_moe"], d_model=320, d_ff=d_ff, d_ff_shared=d_ff_shared, n_experts=E, top_k=k)
    wq = synth.make_weights_q4(cfg) if q4 else None
    w = None if q4 else synth.make_weights(cfg)
    L = Q4Layer(cfg, wq, split, max_tokens=577) if q4 else GpuLayer(cfg, w, split, max_tokens=577)
    try:
        for T in (1, 2, 4, 9, 65, 321, 577):
            print("joint launch E=%d H=%d Hs=%d T=%d" % (E, d_ff, d_ff_shared, T), flush=True)
            xb = synth.make_tokens(cfg, T)
            lg = synth.make_router_logits(cfg, xb)
            if q4:
                yo = oracle.layer_forward_q4(xb, wq, logits=lg, top_k=k)
            else:
                yo = oracle.layer_forward(xb, w["w_gate"], w["w_up"], w["w_down"], logits=lg, top_k=k,
                                          shared=(w["s_gate"], w["s_up"], w["s_down"]))
            if T < 16:
                # fp32 sums of exact products; the host's share splits the activations into two bf16 parts
                assert_parity(L.forward(xb, lg, mode=si.SI_DECODE), yo, tol=1e-4 if split[2] == 0 else 1e-3)
            for n_g in {0, T}:
                assert_parity(L.forward(xb, lg, mode=si.SI_PREFILL, n_g=n_g), yo)
    finally:
        L.close()
