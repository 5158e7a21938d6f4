"""4-bit prompt phase with scales of 2^117 and more, for which 1032 times the scale is no longer a float: such a layer takes
kernels that form code - 8 first.  Scales of three significant bits, so that a weight is a bfloat16; tokens (or, for the down
projection, activations) scaled down by as much."""
import numpy as np
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import assert_parity
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


def _bf16(a):
    return (np.ascontiguousarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _scales(rng, shape, exponent):
    return _bf16(2.0 ** exponent * rng.choice([1.0, 1.25, 1.5, 1.75], size=shape))


# largest scale 1.75 x 2^exponent; 2^117 x 1.75 still fits the ordinary form, 2^124 x 1.75 is the last before 8 x scale overflows
@pytest.mark.parametrize("which", ["gate", "up", "down"])
@pytest.mark.parametrize("exponent", [116, 117, 118, 124])
def test_wide_scales(oracle, which, exponent):
    d_model, d_ff = 192, 320
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff, seed=exponent)
    rng = np.random.default_rng(exponent)
    wq = synth.make_weights_q4(cfg)
    x = rng.standard_normal((300, d_model))
    e = {"gate": -4, "up": -4, "down": -4}
    if which == "down":
        e["up"] = -exponent + 6       # activations of about 2^(6 - exponent)
    else:
        x *= 2.0 ** -exponent
        e["gate"] = e["up"] = exponent - 4
    e[which] = exponent
    for key in e:
        wq["z_" + key] = _scales(rng, wq["z_" + key].shape, e[key])
    xb = _bf16(x)
    yo = oracle.layer_forward_q4(xb, wq)
    L = Q4Layer(cfg, wq, (1.0, 0.0, 0.0), max_tokens=300)
    try:
        for T in (20, 150, 300):
            print("wide scales %s 2^%d T=%d" % (which, exponent, T), flush=True)
            assert_parity(L.forward(xb[:T], None, mode=si.SI_PREFILL), yo[:T])
    finally:
        L.close()


@pytest.mark.parametrize("split,d_ff_shared", [((1.0, 0.0, 0.0), 0), ((0.4, 0.6, 0.0), 256)])
def test_wide_kernels_give_the_same_results(split, d_ff_shared):
    """An expert without rows holds a wide scale (or an infinite one): every other expert's result is bit for bit that of the layer
    without it."""
    cfg = synth.scaled(synth.CONFIGS["qwen_moe"], d_model=192, d_ff=320, d_ff_shared=d_ff_shared, n_experts=4, top_k=2, seed=3)
    wq = synth.make_weights_q4(cfg)
    xb = synth.make_tokens(cfg, 400)
    lg = np.random.default_rng(4).standard_normal((400, 4)).astype(np.float32)
    lg[:, 2] -= 100.0
    outs = []
    for bits in (None, (127 + 120) << 7, 0x7f80):
        w = dict(wq)
        if bits:
            w["z_down"] = wq["z_down"].copy()
            w["z_down"][2, -1, -1] = bits
        L = Q4Layer(cfg, w, split, max_tokens=400)
        try:
            outs.append(L.forward(xb, lg, mode=si.SI_PREFILL))
        finally:
            L.close()
    assert np.all(np.isfinite(outs[0]))
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])
