"""The 4-bit gate/up kernel that splits long rows over the waves of a block, at its edges, against the oracle: the first d_model it takes
and one below it, odd numbers of scale groups and pieces, one to ten column groups a block, 1 to 9 tokens (one pass over the weights and three).  Products are exact and sums fp32: 1e-4 x RMS as for the other
generation-phase kernels."""
import numpy as np
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,d_ff", [(6656, 128), (6720, 64), (6976, 576), (7424, 64), (8128, 192), (8192, 64), (8192, 2304), (6720, 18944), (6720, 6144), (6720, 6208), (6720, 8256)])
def test_split_rows(oracle, d_model, d_ff):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff, seed=300 + d_model)
    wq = synth.make_weights_q4(cfg)
    L = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=16)
    try:
        xp = synth.make_tokens(cfg, 9)
        yo = oracle.layer_forward_q4(xp, wq)
        full = None
        for T in (9, 1, 3, 4, 5):
            print("split rows M=%d H=%d T=%d" % (d_model, d_ff, T), flush=True)
            y = L.forward(xp[:T], None, mode=si.SI_DECODE)
            assert_parity(y, yo[:T], tol=1e-4)
            full = y if full is None else full
            assert np.array_equal(y, full[:T])  # a token's sums do not depend on its batch
    finally:
        L.close()


@pytest.mark.parametrize("d_model,chunks", [(6720, 120), (6720, 140), (8192, 100)])
def test_pieces_of_a_part(d_model, chunks):
    """A streamed part in one launch and in pieces, in a layer of a size for either kernel: the same bits."""
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=64 * chunks, seed=chunks)
    wq = synth.make_weights_q4(cfg)
    xp = synth.make_tokens(cfg, 5)
    for split in ((0.0, 1.0, 0.0), (20 / chunks, 1 - 20 / chunks, 0.0)):
        outs = []
        for stage_mib in (256, 16):
            print("pieces M=%d chunks=%d stage %d MiB" % (d_model, chunks, stage_mib), flush=True)
            L = Q4Layer(cfg, wq, split, max_tokens=8, stage_mib=stage_mib)
            try:
                outs.append([L.forward(xp[:T], None, mode=si.SI_DECODE) for T in (1, 5)])
            finally:
                L.close()
        assert all(np.array_equal(a, b) for a, b in zip(*outs))
