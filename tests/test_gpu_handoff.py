"""The hand-off between GPU and host on both sides of its dispatch line (rows and results up to 256 KB are moved by kernels,
above by the copy engine): split layers with a host part, dense, MoE and shared, repeated calls with other rows and other
X1 / X2 cuts on the same layer, against the oracle."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,d_ff_shared", [(1, 1, 0), (4, 2, 0), (4, 2, 256)])
def test_handoff_sizes(oracle, E, k, d_ff_shared):
    # 512 rows of 256 elements are 256 KB of x (bf16), 256 rows are 256 KB of results (fp32)
    base = synth.CONFIGS["llama2_70b" if E == 1 else "qwen_moe"]
    cfg = synth.scaled(base, d_model=256, d_ff=320, n_experts=E, top_k=k, d_ff_shared=d_ff_shared)
    w = synth.make_weights(cfg)
    shared = (w["s_gate"], w["s_up"], w["s_down"]) if d_ff_shared else None
    L = GpuLayer(cfg, w, (0.4, 0.2, 0.4), max_tokens=600)
    try:
        for T, n_g in ((1, 0), (4, 0), (3, 3), (256, 0), (257, 0), (512, 0), (513, 0), (600, 87), (600, 344), (5, 2), (600, 600)):
            print("hand-off E=%d Hs=%d T=%d n_g=%d" % (E, d_ff_shared, T, n_g), flush=True)
            xb = synth.make_tokens(cfg, T, stream=T + n_g)
            lg = synth.make_router_logits(cfg, xb)
            yo = oracle.layer_forward(xb, w["w_gate"], w["w_up"], w["w_down"], logits=lg, top_k=k, shared=shared)
            assert_parity(L.forward(xb, lg, n_g=n_g), yo)
    finally:
        L.close()


def test_handoff_ms_is_the_wait():
    """handoff_ms is what the host waits for the assignment, not the time it spends enqueuing the resident part: a 4-bit layer
    whose prompt phase goes through a one-chunk bf16 scratch enqueues 174 resident launches between the hand-off kernel and the
    wait, by whose end the assignment has long arrived (measured: 1 us; with the launches counted, 400)."""
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=4096, d_ff=4096)
    L = Q4Layer(cfg, synth.make_weights_q4(cfg), (0.9, 0.0, 0.1), max_tokens=4, deq_mib=1)
    try:
        x = synth.make_tokens(cfg, 4)
        waits = []
        for _ in range(20):
            L.forward(x, None, mode=si.SI_PREFILL)
            st = si.si_layer_stats(L.h)
            waits.append(st["handoff_ms"])
            assert st["handoff_ms"] <= st["enqueue_ms"]
        print("hand-off waits (ms): min %.4f median %.4f" % (min(waits), sorted(waits)[10]), flush=True)
        assert min(waits) < 0.05
    finally:
        L.close()
