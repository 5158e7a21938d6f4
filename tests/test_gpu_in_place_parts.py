"""Streamed parts of dense layers that the generation-phase kernels read from host memory in the launches of the resident part, on both sides
of the lines (2 MB, 8 MB where the host computes a share, 4 tokens; parts of up to 8 chunks, a slot each, and more): against the oracle, and
bit for bit against the same call with profiling on, which copies the part in launches of its own; recorded calls too."""
import numpy as np
import pytest
import torch

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer, assert_parity

pytestmark = pytest.mark.gpu


# chunks of 64 columns: 96 KiB at d_model 256, 384 KiB at 1024, 768 KiB at 2048
@pytest.mark.parametrize("d_model,chunks,cg,cc", [(256, 11, 3, 3), (256, 40, 21, 0), (256, 40, 22, 0), (320, 9, 8, 0), (1024, 24, 9, 2), (1024, 24, 5, 0),
                                                  (1024, 24, 6, 0), (2048, 24, 10, 1), (2048, 24, 11, 1), (64, 3, 1, 1)])
def test_in_place(oracle, d_model, chunks, cg, cc):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=64 * chunks, seed=chunks + cg)
    w = synth.make_weights(cfg)
    L = GpuLayer(cfg, w, ((chunks - cg - cc) / chunks, cg / chunks, cc / chunks), max_tokens=8)
    try:
        for T in (1, 2, 3, 4, 5, 1):
            print("in place M=%d chunks=%d cg=%d cc=%d T=%d" % (d_model, chunks, cg, cc, T), flush=True)
            x = synth.make_tokens(cfg, T, stream=T)
            yo = oracle.layer_forward(x, w["w_gate"], w["w_up"], w["w_down"])
            y = L.forward(x, None, mode=si.SI_DECODE)
            assert_parity(y, yo, tol=1e-3 if cc else 1e-4)  # (the host's share splits the activations into two bf16 parts)
            si.si_layer_set_profiling(L.h, 1)
            assert np.array_equal(L.forward(x, None, mode=si.SI_DECODE), y)
            si.si_layer_set_profiling(L.h, 0)
            assert_parity(L.forward(x, None, n_g=T, mode=si.SI_DECODE), yo, tol=1e-4)  # CG' on the GPU
    finally:
        L.close()


def test_recorded():
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=512, d_ff=1024, seed=8)
    L = GpuLayer(cfg, synth.make_weights(cfg), (0.5, 0.5, 0.0), max_tokens=4)  # (8 chunks of 192 KiB)
    x = torch.zeros((4, 512), dtype=torch.int16, device="cuda:0")
    y, eager = (torch.empty((4, 512), dtype=torch.float32, device="cuda:0") for _ in range(2))

    def call(out):
        si.si_layer_forward(L.h, x.data_ptr(), None, 4, 0, si.SI_DECODE, out.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)

    try:
        x.copy_(torch.from_numpy(synth.make_tokens(cfg, 4).view("int16")))
        call(eager)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call(y)
        for r in range(4):
            x.copy_(torch.from_numpy(synth.make_tokens(cfg, 4, stream=2 + r).view("int16")))
            y.zero_()
            g.replay()
            call(eager)
            torch.cuda.synchronize()
            assert float(eager.abs().max()) > 0 and torch.equal(y, eager), r
    finally:
        L.close()
