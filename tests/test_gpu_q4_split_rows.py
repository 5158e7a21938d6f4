"""The 4-bit gate/up kernel that splits long rows over the waves of a block, at its edges, against the oracle: the first d_model it takes
and one below it, odd numbers of scale groups and pieces, one to ten column groups a block and more than LDS holds at once, 1 to 9 tokens
(one pass over the weights and three); parts of experts, rows that start after others, tokens by a table.  Products are exact and sums fp32: 1e-4 x RMS as
for the other generation-phase kernels."""
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


def test_more_groups_than_lds_holds(oracle):
    """12816 groups of 4 columns on 512 blocks: 25 or 26 each, of which LDS holds 25 at d_model 8192, so that some blocks take a second
    stretch (the next one's scales and sums in the place of the first's), for two passes over the rows."""
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=8192, d_ff=64 * 801, seed=801)
    wq = synth.make_weights_q4(cfg, threads=16)
    L = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=8)
    try:
        xp = synth.make_tokens(cfg, 5)
        print("stretches T=5", flush=True)
        y = L.forward(xp, None, mode=si.SI_DECODE)
        sel = np.array([0, 4], np.int32)
        assert_parity(y[sel], oracle.layer_forward_q4(xp, wq, sel=sel), tol=1e-4)
        for T in (1, 4):
            print("stretches T=%d" % T, flush=True)
            assert np.array_equal(L.forward(xp[:T], None, mode=si.SI_DECODE), y[:T])
    finally:
        L.close()


# (experts, top-k, d_ff, d_ff_shared, split): all three parts; streamed experts and a streamed shared one; a resident shared expert of 2 chunks
# beside routed ones without a resident part
@pytest.mark.parametrize("d_model", [6720, 8192])
@pytest.mark.parametrize("E,k,d_ff,d_ff_shared,split", [(1, 1, 704, 0, (0.4, 0.3, 0.3)), (4, 2, 192, 0, (1 / 3, 1 / 3, 1 / 3)), (4, 2, 192, 128, (0.0, 1.0, 0.0)),
                                                        (4, 2, 64, 320, (0.4, 0.6, 0.0))])
def test_parts_and_experts(oracle, d_model, E, k, d_ff, d_ff_shared, split):
    cfg = synth.scaled(synth.CONFIGS["qwen_moe" if E > 1 else "llama2_70b"], d_model=d_model, d_ff=d_ff, d_ff_shared=d_ff_shared, n_experts=E, top_k=k, seed=d_model + d_ff)
    wq = synth.make_weights_q4(cfg)
    L = Q4Layer(cfg, wq, split, max_tokens=16)
    try:
        for T in (1, 3, 9):
            xp = synth.make_tokens(cfg, T, stream=T)
            lg = synth.make_router_logits(cfg, xp)
            yo = oracle.layer_forward_q4(xp, wq, logits=lg, top_k=k)
            for n_g in sorted({0, T // 2, T}):
                print("parts M=%d E=%d H=%d+%d T=%d n_g=%d" % (d_model, E, d_ff, d_ff_shared, T, n_g), flush=True)
                y = L.forward(xp, lg, n_g=n_g, mode=si.SI_DECODE)
                n_x1 = T - n_g if split[2] else 0  # rows with a share of the host's, which takes the activations as two bf16 parts
                if n_x1:
                    assert_parity(y[:n_x1], yo[:n_x1])
                if n_x1 < T:
                    assert_parity(y[n_x1:], yo[n_x1:], tol=1e-4)
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
