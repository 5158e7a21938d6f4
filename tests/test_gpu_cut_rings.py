"""Rings of the prompt-phase tiles that are cut along their columns (a launch of few tiles; up to 160 rows): bodies of 64, 96, 128
and 160 rows have rings of 4, 4, 4 and 3 stages of weights (of rows 3, 4, 4 and 3), so each runs here with fewer k-tiles than stages, as many and more: d_model / 64 in
FC1, and in FC2 the chunks of one of four k-splits, two of which differ by one."""
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity

pytestmark = pytest.mark.gpu

ROWS = (33, 64, 65, 96, 97, 128, 129, 160)


@pytest.mark.parametrize("k_tiles,chunks", [(1, 14), (2, 18), (3, 22), (4, 5), (5, 10), (6, 27), (7, 16), (11, 33)])
def test_cut_tiles(oracle, k_tiles, chunks):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=64 * k_tiles, d_ff=64 * chunks, seed=800 + k_tiles)
    w = synth.make_weights(cfg)
    xp = synth.make_tokens(cfg, max(ROWS))
    yo = oracle.layer_forward(xp, w["w_gate"], w["w_up"], w["w_down"])
    L = GpuLayer(cfg, w, (1.0, 0.0, 0.0), max_tokens=max(ROWS))
    try:
        for T in ROWS:
            print("k-tiles %d chunks %d T %d" % (k_tiles, chunks, T), flush=True)
            assert_parity(L.forward(xp[:T], None, mode=si.SI_PREFILL), yo[:T])
    finally:
        L.close()
