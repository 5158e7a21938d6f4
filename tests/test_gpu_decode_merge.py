"""The generation-phase merge over more terms than it has waves (one to three batches, the last one partly filled), with and
without a shared expert, at widths that fill its lanes in part and over several blocks; layer resident and split.  Against the
oracle: exact products, fp32 sums: 1e-4 x RMS,
1e-3 with a part on the host."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("place", [(1.0, 0.0, 0.0), (0.4, 0.3, 0.3)])
@pytest.mark.parametrize("k,d_ff_shared", [(3, 0), (7, 256), (8, 256), (16, 0), (20, 128)])
@pytest.mark.parametrize("d_model", [64, 192, 320])
def test_merge_terms(oracle, d_model, k, d_ff_shared, place):
    cfg = synth.scaled(synth.CONFIGS["qwen_moe"], d_model=d_model, d_ff=128, d_ff_shared=d_ff_shared, n_experts=24, top_k=k, seed=40 + k)
    w = synth.make_weights(cfg)
    L = GpuLayer(cfg, w, place, max_tokens=4)
    try:
        for T in (1, 3):
            xb = synth.make_tokens(cfg, T)
            lg = synth.make_router_logits(cfg, xb)
            sh = (w["s_gate"], w["s_up"], w["s_down"]) if d_ff_shared else None
            yo = oracle.layer_forward(xb, w["w_gate"], w["w_up"], w["w_down"], logits=lg, top_k=k, shared=sh)
            # (the host's share splits the activations into two bf16 parts)
            assert_parity(L.forward(xb, lg, mode=si.SI_DECODE), yo, tol=1e-4 if place[2] == 0 else 1e-3)
    finally:
        L.close()


@pytest.mark.parametrize("k,d_ff_shared", [(1, 0), (3, 512), (4, 0), (5, 512), (9, 128)])
def test_prompt_merge_terms(oracle, k, d_ff_shared):
    """The prompt-phase merge, four terms at a time, over one to four slabs of each kind; bf16 activations: the usual tolerance."""
    cfg = synth.scaled(synth.CONFIGS["qwen_moe"], d_model=320, d_ff=512, d_ff_shared=d_ff_shared, n_experts=12, top_k=k, seed=60 + k)
    w = synth.make_weights(cfg)
    L = GpuLayer(cfg, w, (1.0, 0.0, 0.0), max_tokens=64)
    try:
        for T in (3, 64):
            xp = synth.make_tokens(cfg, T)
            lg = synth.make_router_logits(cfg, xp)
            sh = (w["s_gate"], w["s_up"], w["s_down"]) if d_ff_shared else None
            yo = oracle.layer_forward(xp, w["w_gate"], w["w_up"], w["w_down"], logits=lg, top_k=k, shared=sh)
            assert_parity(L.forward(xp, lg, mode=si.SI_PREFILL), yo)
    finally:
        L.close()
