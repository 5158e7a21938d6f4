"""Generation calls of dense layers with a streamed part and nothing on the host, recorded into a HIP graph: eagerly such a part may
travel on the copy stream, recorded a kernel copies it in the call's own stream.  Several replays with eager calls in between, bit for
bit the eager results."""
import pytest
import torch

import paper_2411_15715_amd as si
import synth
from gpu_helpers import GpuLayer
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,d_model,d_ff,split,T,n_g,stage_mib", [
    ("bf16", 1024, 1024, (0.5, 0.5, 0.0), 8, 0, 0), ("bf16", 1024, 1024, (0.25, 0.75, 0.0), 1, 0, 1),
    ("bf16", 4096, 1536, (0.125, 0.875, 0.0), 4, 0, 4), ("bf16", 512, 1536, (0.25, 0.25, 0.5), 3, 3, 0),
    ("q4", 1024, 2048, (0.5, 0.5, 0.0), 8, 0, 0)])
def test_replays(form, d_model, d_ff, split, T, n_g, stage_mib):
    cfg = synth.scaled(synth.CONFIGS["llama2_70b"], d_model=d_model, d_ff=d_ff, seed=d_ff)
    L = GpuLayer(cfg, synth.make_weights(cfg), split, max_tokens=16, stage_mib=stage_mib) if form == "bf16" else \
        Q4Layer(cfg, synth.make_weights_q4(cfg), split, max_tokens=16, stage_mib=stage_mib)
    dev = torch.device("cuda:0")
    x = torch.zeros((T, d_model), dtype=torch.int16, device=dev)
    y, eager = (torch.empty((T, d_model), dtype=torch.float32, device=dev) for _ in range(2))

    def call(out):
        si.si_layer_forward(L.h, x.data_ptr(), None, T, n_g, si.SI_DECODE, out.data_ptr(), stream=torch.cuda.current_stream().cuda_stream)

    try:
        x.copy_(torch.from_numpy(synth.make_tokens(cfg, T).view("int16")))
        call(eager)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call(y)
        for r in range(4):
            print("replay %d of %s M=%d H=%d T=%d" % (r, form, d_model, d_ff, T), flush=True)
            x.copy_(torch.from_numpy(synth.make_tokens(cfg, T, stream=2 + r).view("int16")))
            y.zero_()
            g.replay()
            if r % 2:
                torch.cuda.synchronize()
            call(eager)
            torch.cuda.synchronize()
            assert torch.isfinite(eager).all() and float(eager.abs().max()) > 0
            assert torch.equal(y, eager), r
    finally:
        L.close()
