"""Prompt calls recorded into a HIP graph: the launches of a call take their tiles from counters on the device, so every replay has to
start with them clear.  Launches of several rounds of tiles, several replays with eager prompt and generation calls and
synchronisations in between; each result bit for bit the eager one."""
import numpy as np
import pytest
import torch

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["bf16", "q4"])
@pytest.mark.parametrize("E,k,d_ff,d_ff_shared", [(1, 1, 17408, 0), (8, 2, 2560, 0), (8, 2, 1280, 5120)])
def test_replays(form, E, k, d_ff, d_ff_shared):
    base = synth.CONFIGS["qwen_moe" if E > 1 else "llama2_70b"]
    cfg = synth.scaled(base, d_model=512, d_ff=d_ff, d_ff_shared=d_ff_shared, n_experts=E, top_k=k, seed=80 + E)
    L = GpuLayer(cfg, synth.make_weights(cfg), (1.0, 0.0, 0.0), max_tokens=700) if form == "bf16" else \
        Q4Layer(cfg, synth.make_weights_q4(cfg), (1.0, 0.0, 0.0), max_tokens=700)
    dev = torch.device("cuda:0")
    T = 700
    x = torch.zeros((T, 512), dtype=torch.int16, device=dev)
    lg = torch.zeros((T, E), dtype=torch.float32, device=dev)
    y = torch.empty((T, 512), dtype=torch.float32, device=dev)

    def call(out, n=T, mode=si.SI_PREFILL):
        si.si_layer_forward(L.h, x.data_ptr(), lg.data_ptr() if E > 1 else None, n, 0, mode, out.data_ptr(),
                            stream=torch.cuda.current_stream().cuda_stream)

    def inputs(seed):
        xb = synth.make_tokens(cfg, T, stream=seed)
        x.copy_(torch.from_numpy(xb.view(np.int16)))
        if E > 1:
            lg.copy_(torch.from_numpy(synth.make_router_logits(cfg, xb)))

    try:
        inputs(1)
        call(y)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call(y)
        eager = torch.empty_like(y)
        for r in range(4):
            print("replay %d of %s E=%d H=%d" % (r, form, E, d_ff), flush=True)
            inputs(2 + r)
            y.zero_()
            g.replay()
            if r % 2:
                torch.cuda.synchronize()
                call(eager, 3, si.SI_DECODE)
            call(eager)
            torch.cuda.synchronize()
            assert torch.isfinite(eager).all() and float(eager.abs().max()) > 0
            assert torch.equal(y, eager), r
    finally:
        L.close()
