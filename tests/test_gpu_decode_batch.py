"""Generation phase: a token's result does not depend on the batch it is in (the cuts of all sums follow from the layer's shape):
every row of a call of several tokens equals, bit for bit, the call of that token alone.  Layers on both sides of the line up
to which the resident part is cut into more slots, bf16 and 4-bit, with and without a shared expert."""
import numpy as np
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,d_ff,E,k,d_ff_shared,q4", [
    (4096, 576, 12, 2, 0, False), (512, 1088, 6, 3, 256, False), (4096, 1088, 4, 4, 0, False), (3328, 2240, 1, 1, 0, False),
    (1024, 576, 8, 2, 320, True)])
def test_batch_independent(d_model, d_ff, E, k, d_ff_shared, q4):
    base = synth.CONFIGS["qwen_moe" if d_ff_shared else "llama2_70b" if E == 1 else "mixtral_8x7b"]
    cfg = synth.scaled(base, d_model=d_model, d_ff=d_ff, n_experts=E, top_k=k, d_ff_shared=d_ff_shared)
    split = (1.0, 0.0, 0.0)
    L = Q4Layer(cfg, synth.make_weights_q4(cfg), split, max_tokens=16) if q4 else GpuLayer(cfg, synth.make_weights(cfg), split, max_tokens=16)
    try:
        x = synth.make_tokens(cfg, 16)
        lg = synth.make_router_logits(cfg, x)
        row = lambda a, i, j: None if a is None else a[i:j]
        alone = np.concatenate([L.forward(x[t:t + 1], row(lg, t, t + 1), mode=si.SI_DECODE) for t in range(16)])
        for T in (2, 3, 4, 7, 16):
            print("batch M=%d H=%d E=%d T=%d" % (d_model, d_ff, E, T), flush=True)
            assert np.array_equal(L.forward(x[:T], row(lg, 0, T), mode=si.SI_DECODE), alone[:T]), T
    finally:
        L.close()
