"""Rings of the 4-bit prompt-phase GEMMs: one to eighteen k-tiles of FC1 (blocks of codes of four k-tiles, full and partial, rows of scales
that start at odd places) and of FC2 (one chunk a block), against the oracle and, bit for bit, against the GEMMs on weights that a kernel of its own has
made bf16: the same products in the same order.  A launch of few tiles cuts those of more than 64 rows along their rows, so the first test runs bodies of up to
128 rows; the second has 17 tiles and more for each XCD, which are whole: every body of 32 to 256 rows and a second pass over the rows of a last tile beyond
256, on scales of eight bits, where converting a weight rounds it."""
import numpy as np
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k_tiles,d_ff", [(1, 192), (2, 640), (3, 576), (4, 128), (5, 448), (6, 832), (7, 64), (8, 512), (9, 1088), (10, 256), (11, 704),
                                          (12, 384), (13, 960), (17, 320), (18, 1152)])
def test_blocks_of_codes(oracle, k_tiles, d_ff):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=64 * k_tiles, d_ff=d_ff, seed=70 + k_tiles)
    wq = synth.make_weights_q4(cfg)
    # Scales of three significant bits: a weight then has at most 7 and is a bfloat16.  Otherwise each of the three weights and the
    # activation of a product is rounded by up to 2^-9, 2.3e-3 (rms) of a product in all, which over the 64 products of the smallest sum
    # and 112 000 results exceeds 2e-2 of the RMS once (both ways of the comparison alike); with the activation alone it is half of that.
    for key in ("z_gate", "z_up", "z_down"):
        wq[key] = (wq[key] & 0xFF80) | 0x20
    xp = synth.make_tokens(cfg, 250)
    yo = oracle.layer_forward_q4(xp, wq)
    one, two = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=250), Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=250, deq_mib=64)
    try:
        for T in (10, 50, 97, 150, 200, 250):
            print("k-tiles %d d_ff %d T %d" % (k_tiles, d_ff, T), flush=True)
            y = one.forward(xp[:T], None, mode=si.SI_PREFILL)
            assert_parity(y, yo[:T])
            assert np.array_equal(y, two.forward(xp[:T], None, mode=si.SI_PREFILL))
    finally:
        one.close()
        two.close()


# FC1: 136 column tiles, one to nine and eighteen k-tiles.  FC2: 32 column tiles of three experts (every token takes all of them) in two k-splits of none
# to nine and eighteen chunks, mostly of two lengths.
@pytest.mark.parametrize("E,k_tiles,chunks", [(1, k, 272) for k in (1, 2, 3, 4, 5, 6, 7, 8, 9, 18)] + [(3, 128, c) for c in (1, 3, 5, 7, 9, 11, 13, 15, 17, 36)])
def test_whole_tiles(oracle, E, k_tiles, chunks):
    cfg = synth.scaled(synth.CONFIGS["mixtral_8x7b" if E > 1 else "llama2_70b"], d_model=64 * k_tiles, d_ff=64 * chunks, n_experts=E, top_k=E, seed=500 + k_tiles + chunks)
    wq = synth.make_weights_q4(cfg)
    xp = synth.make_tokens(cfg, 300)
    lg = synth.make_router_logits(cfg, xp)
    sel = np.array([0, 9, 31, 250, 299], np.int32)
    yo = oracle.layer_forward_q4(xp, wq, logits=lg, top_k=E, sel=sel)
    one, two = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=300), Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=300, deq_mib=512)
    try:
        for T in (20, 50, 80, 110, 150, 180, 210, 250, 300):
            print("whole tiles, experts %d k-tiles %d chunks %d T %d" % (E, k_tiles, chunks, T), flush=True)
            lt = lg[:T] if E > 1 else None
            y = one.forward(xp[:T], lt, mode=si.SI_PREFILL)
            assert np.array_equal(y, two.forward(xp[:T], lt, mode=si.SI_PREFILL))
        assert_parity(y[sel], yo)
    finally:
        one.close()
        two.close()
