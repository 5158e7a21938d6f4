"""Small calls of split layers on both sides of their dispatch lines, against the oracle: parts that a kernel copies in the
caller's stream (dense up to 32 MB where the host computes a share, else up to 8 MB, of several experts up to 4 MB, both with few
rows) or the copy stream does, a host share that the calling thread runs itself or the workers do, streamed parts of up to 8
chunks (a slot each) and more; calls in a row on one layer."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,d_model,d_ff,split", [
    (1, 1, 64, 192, (1 / 3, 1 / 3, 1 / 3)), (1, 1, 256, 704, (0.4, 0.3, 0.3)), (1, 1, 320, 1216, (0.1, 0.45, 0.45)),
    (1, 1, 448, 1088, (0.0, 0.5, 0.5)), (1, 1, 1024, 1472, (0.3, 0.3, 0.4)),
    (4, 2, 2048, 768, (0.5, 5 / 12, 1 / 12)), (4, 2, 2048, 768, (0.5, 0.5, 0.0)), (3, 1, 192, 640, (0.2, 0.5, 0.3))])
def test_small_split(oracle, E, k, d_model, d_ff, split):
    cfg = synth.scaled(synth.CONFIGS["mixtral_8x7b" if E > 1 else "llama2_70b"], d_model=d_model, d_ff=d_ff, n_experts=E, top_k=k, seed=d_ff)
    w = synth.make_weights(cfg)
    L = GpuLayer(cfg, w, split, max_tokens=16)
    try:
        for T in (1, 4, 8, 2, 16, 1):
            print("small split E=%d M=%d H=%d T=%d" % (E, d_model, d_ff, T), flush=True)
            x = synth.make_tokens(cfg, T, stream=T)
            lg = synth.make_router_logits(cfg, x)
            yo = oracle.layer_forward(x, w["w_gate"], w["w_up"], w["w_down"], logits=lg, top_k=k)
            # fp32 sums of exact products; the host's share splits the activations into two bf16 parts
            assert_parity(L.forward(x, lg, mode=si.SI_DECODE), yo, tol=1e-3)
            assert_parity(L.forward(x, lg, n_g=T, mode=si.SI_DECODE), yo, tol=1e-3)
    finally:
        L.close()


@pytest.mark.parametrize("chunks,cg,cc,T", [(24, 21, 1, 3), (24, 22, 1, 3), (12, 5, 0, 1), (12, 6, 0, 1), (12, 5, 0, 2)])
def test_one_part_sizes(oracle, chunks, cg, cc, T):
    """One dense part (chunks of 1.5 MB) just below and just above 32 MB beside a host share; just below and just above 8 MB without one, and
    below with a row too many."""
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=4096, d_ff=64 * chunks, seed=5)
    w = synth.make_weights(cfg)
    x = synth.make_tokens(cfg, T)
    yo = oracle.layer_forward(x, w["w_gate"], w["w_up"], w["w_down"])
    L = GpuLayer(cfg, w, ((chunks - cg - cc) / chunks, cg / chunks, cc / chunks), max_tokens=3)
    try:
        for _ in range(3):
            assert_parity(L.forward(x, None), yo, tol=1e-3 if cc else 1e-4)
    finally:
        L.close()
