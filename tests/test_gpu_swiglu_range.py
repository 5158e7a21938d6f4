"""SiLU(gate) * up of the prompt phase over the whole range in which exp(-gate) is finite, with bf16 and 4-bit weights: gate
values down to -88.5, whose SiLU (-3e-37) is a normal fp32 number although its reciprocal factor is not, made visible by an
up value of 2^60 and passed through a unit down projection.  One rounding to bf16 and 1e-5 of the exponential: 2^-8."""
import numpy as np
import pytest

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q4", [False, True])
def test_swiglu_range(q4):
    n = 256
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=n, d_ff=n)
    bf16 = lambda a: (np.ascontiguousarray(a, np.float32).view(np.uint32) >> 16).astype(np.uint16)  # (of values that are bf16)
    z = np.concatenate([-88.5 + 0.5 * np.arange(n // 2), 0.25 * np.arange(n // 2)]).astype(np.float32)
    z = (bf16(z).astype(np.uint32) << 16).view(np.float32)
    up = 2.0 ** 60
    if q4:
        codes = np.full((n, n), 8, np.uint8)
        codes[:, 0] = 9  # weight 1 * scale at element 0 of every row
        eye = np.where(np.eye(n) > 0, 9, 8).astype(np.uint8)
        pack = lambda q: (q[:, 0::2] | (q[:, 1::2] << 4)).astype(np.uint8)[None]
        scale = lambda v: bf16(np.repeat(np.reshape(v, (n, 1)), n // 64, axis=1))[None]
        L = Q4Layer(cfg, {"q_gate": pack(codes), "q_up": pack(codes), "q_down": pack(eye), "z_gate": scale(z), "z_up": scale(np.full(n, up)),
                          "z_down": bf16(np.ones((1, n // 64, n)))}, (1.0, 0.0, 0.0), max_tokens=64)
    else:
        col = lambda v: np.concatenate([np.reshape(v, (n, 1)), np.zeros((n, n - 1))], axis=1)
        L = GpuLayer(cfg, {"w_gate": bf16(col(z))[None], "w_up": bf16(col(np.full(n, up)))[None], "w_down": bf16(np.eye(n))[None]},
                     (1.0, 0.0, 0.0), max_tokens=64)
    try:
        x = np.zeros((40, n), np.float32)
        x[:, 0] = 1.0
        y = L.forward(bf16(x), None, mode=si.SI_PREFILL).astype(np.float64)
        ref = z.astype(np.float64) / (1.0 + np.exp(-z.astype(np.float64))) * up
        assert np.all(np.abs(y - ref) <= 2.0 ** -8 * np.abs(ref)), float(np.max(np.abs(y / np.where(ref == 0, 1, ref) - 1)))
    finally:
        L.close()
