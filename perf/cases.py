"""Performance cases of the partitioned FFN / MoE layer, called as a serving program calls it.

A serving program creates a layer once (weights, slicing rates, workspaces) and then runs forward calls on it:
generation-phase calls with one or a few tokens, batches of a few dozen sequences, prompts of hundreds to thousands of
tokens.  prepare() makes the layer and one call's inputs, run() is one si_layer_forward (or si_stack_forward) call.
The shapes of the listed cases are the workload shapes of this repository's benchmark (synth.CONFIGS); draw() spreads
over the ranges between and around them.

A case is a dict:
  dtype     "bf16" or "q4" (4-bit codes with bf16 group scales)
  d_model, d_ff, n_experts, top_k, d_ff_shared   layer shape (n_experts == 1: dense MLP; d_ff_shared == 0: no shared expert)
  router    "none" (dense), "gate" (logits ~ N(0, 1)) or "zipf" (the same plus a -1.1 ln(rank) popularity bias)
  tokens    rows of x
  n_g       trailing tokens whose CC share runs on the GPU (prompt phase of a layer with a CC part)
  r_gg, r_cg, r_cc   slicing rates: resident / streamed over the host link / computed on the host
  layers    1: one layer; more: a stack of that many layers with the residual connection between them
"""
import math

import numpy as np
import torch

import paper_2411_15715_amd as si

W_STD = 0.02
GROUP = 64            # weights per scale of the 4-bit form
POOL_ELEMS = 1 << 30  # random weights shared by all layers: gate, up and down are windows of it
POOL_CODES = 1 << 28  # the same for packed 4-bit codes (bytes)
MAX_FLOPS = 6.0 * 8192 * 16384 * 6144  # the largest listed prompt


def _case(name, **kw):
    c = {"dtype": "bf16", "d_model": 4096, "d_ff": 14336, "n_experts": 1, "top_k": 1, "d_ff_shared": 0, "router": "none",
         "tokens": 1, "n_g": 0, "r_gg": 1.0, "r_cg": 0.0, "r_cc": 0.0, "layers": 1}
    c.update(kw)
    if name:
        c["name"] = name
    return c


MIXTRAL_8X7B = dict(d_model=4096, d_ff=14336, n_experts=8, top_k=2, router="gate")
MIXTRAL_8X22B = dict(d_model=6144, d_ff=16384, n_experts=8, top_k=2, router="gate")
LLAMA2_70B = dict(d_model=8192, d_ff=28672)
QWEN_MOE = dict(d_model=3584, d_ff=2560, n_experts=64, top_k=8, d_ff_shared=20480, router="zipf")
PHIMOE = dict(d_model=4096, d_ff=6400, n_experts=16, top_k=2, router="gate")


def listed():
    return [
        # the smallest call: a tiny layer with all three parts, where launches, copies and host hand-offs are everything
        _case("tiny_split_decode_4", d_model=256, d_ff=704, tokens=4, r_gg=0.4, r_cg=0.3, r_cc=0.3),
        # token-by-token generation on a fine-grained MoE layer: the shortest full-size call
        _case("phimoe_decode_1", tokens=1, **PHIMOE),
        # generation for a few sequences: many small experts and a large shared one
        _case("qwen_moe_decode_4", tokens=4, **QWEN_MOE),
        # generation through consecutive dense layers with their residual connections
        _case("llama2_70b_stack2_decode_1", tokens=1, layers=2, **LLAMA2_70B),
        # a batch of sequences in generation (continuous batching): few rows per expert, every expert used
        _case("mixtral_8x7b_batch_24", tokens=24, **MIXTRAL_8X7B),
        # prompts: bound by weight traffic (about 128 rows per expert) ...
        _case("mixtral_8x7b_prefill_512", tokens=512, **MIXTRAL_8X7B),
        # ... by the matrix cores on a dense layer ...
        _case("llama2_70b_prefill_1024", tokens=1024, **LLAMA2_70B),
        # ... over many experts of very different popularity, a batch of ragged length ...
        _case("qwen_moe_prefill_2011", tokens=2011, **QWEN_MOE),
        # ... and the largest layer and prompt
        _case("mixtral_8x22b_prefill_4096", tokens=4096, **MIXTRAL_8X22B),
        # 4-bit weights, generation for three sequences on a dense layer
        _case("llama2_70b_q4_decode_3", dtype="q4", tokens=3, **LLAMA2_70B),
        # 4-bit weights, an odd prompt length
        _case("mixtral_8x7b_q4_prefill_777", dtype="q4", tokens=777, **MIXTRAL_8X7B),
        # the method's own setting: a layer that does not fit the GPU, half of it streamed and a fifth on the host
        _case("llama2_70b_30_50_20_decode_1", tokens=1, r_gg=0.3, r_cg=0.5, r_cc=0.2, **LLAMA2_70B),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: generation calls, batches, prompts and split layers, dense and MoE, bf16 and 4-bit."""
    kind = rng.choices(["decode", "batch", "prefill", "split"], [0.33, 0.17, 0.4, 0.1])[0]
    q4 = rng.random() < 0.25
    dense = rng.random() < 0.35
    M = 256 * rng.randint(4, 32)
    E = 1 if dense else rng.choice([4, 8, 12, 16, 32, 60, 64])
    k = 1 if dense else rng.randint(1, min(8, E // 2))
    h_max = min(28672, (1 << 29) // (E * M))
    H = max(512, 64 * (_log_int(rng, 1024, max(1024, h_max)) // 64))
    Hs = 0
    if not dense and rng.random() < 0.3:
        Hs = 64 * (_log_int(rng, 1024, 20480) // 64)
    T = {"decode": rng.randint(1, 8), "batch": rng.randint(9, 64)}.get(kind) or _log_int(rng, 65, 4096)
    c = _case(None, dtype="q4" if q4 else "bf16", d_model=M, d_ff=H, n_experts=E, top_k=k, d_ff_shared=Hs,
              router="none" if dense else rng.choice(["gate", "zipf"]), tokens=T)
    if kind == "split":
        c["tokens"] = T = rng.choice([1, 2, 4, _log_int(rng, 65, 1024)])
        c["r_gg"], c["r_cg"], c["r_cc"] = rng.choice([(0.8, 0.2, 0.0), (0.6, 0.3, 0.1), (0.5, 0.5, 0.0), (0.4, 0.4, 0.2)])
        if T > 64 and c["r_cc"] > 0:
            c["n_g"] = T
        # streamed weights cross the host link: at most what the listed split case streams
        cap = 3 * 8192 * 28672 // 2
        while _weights(c, 1.0) * (c["r_cg"] + (c["r_cc"] if c["n_g"] else 0.0)) > cap and c["d_ff"] > 512:
            c["d_ff"] = max(512, c["d_ff"] // 128 * 64)
    if kind == "decode" and rng.random() < 0.2:
        c["layers"] = 2
    while work(c)["flops"] > MAX_FLOPS:
        c["tokens"] = c["tokens"] * 3 // 4
        c["n_g"] = min(c["n_g"], c["tokens"])
    return c


# ------------------------------------------------------------------------------------------------ inputs
_pools = {}


def _pool(kind):
    """Random storage that every layer's weights are windows of (drawn once per process, on the GPU)."""
    if kind not in _pools:
        g = torch.Generator(device="cuda").manual_seed(20241115)
        n = POOL_ELEMS if kind == "bf16" else POOL_CODES
        out = np.empty(n, np.uint16 if kind == "bf16" else np.uint8)
        step = 1 << 26
        for i in range(0, n, step):
            if kind == "bf16":
                v = torch.randn(step, generator=g, device="cuda").mul_(W_STD).to(torch.bfloat16).view(torch.int16)
                out[i:i + step] = v.cpu().numpy().view(np.uint16)
            else:
                # codes of a bell-shaped weight distribution, two to a byte
                q = (torch.randn(2, step, generator=g, device="cuda") * 2.4).round_().add_(8).clamp_(0, 15).to(torch.uint8)
                out[i:i + step] = (q[0] | (q[1] << 4)).cpu().numpy()
        _pools[kind] = out
    return _pools[kind]


def _window(kind, rng, shape):
    p, n = _pool(kind), int(np.prod(shape))
    start = int(rng.integers(0, (p.size - n) // 64 + 1)) * 64
    return p[start:start + n].reshape(shape)


def _scales(rng, shape):
    v = torch.from_numpy(rng.uniform(0.7, 1.3, size=shape).astype(np.float32) * np.float32(W_STD / 2.4))
    return np.ascontiguousarray(v.to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16))


class State:
    """One call's inputs and the layers it runs on."""

    def __init__(self):
        self.layers, self.stack = [], None

    def __del__(self, stack_destroy=si.si_stack_destroy, layer_destroy=si.si_layer_destroy):
        if self.stack is not None:
            stack_destroy(self.stack)
        for h in self.layers:
            layer_destroy(h)


def _make_layer(case, rng):
    M, H, E, Hs = case["d_model"], case["d_ff"], case["n_experts"], case["d_ff_shared"]
    rates = (case["r_gg"], case["r_cg"], case["r_cc"])
    max_tokens = max(64, case["tokens"])
    if case["dtype"] == "q4":
        w = {}
        for pre, lead, h in (("", (E,), H), ("s", (), Hs)):
            if h:
                for n in ("gate", "up", "down"):
                    w["%sq_%s" % (pre, n)] = _window("q4", rng, lead + (h, M // 2))
                w[pre + "z_gate"], w[pre + "z_up"] = (_scales(rng, lead + (h, M // GROUP)) for _ in range(2))
                w[pre + "z_down"] = _scales(rng, lead + (h // GROUP, M))
        return si.si_layer_create_q4(M, H, E, case["top_k"], w, *rates, max_tokens, d_ff_shared=Hs)
    w = [_window("bf16", rng, (E, H, M)) for _ in range(3)]
    shared = tuple(_window("bf16", rng, (Hs, M)) for _ in range(3)) if Hs else None
    return si.si_layer_create(M, H, E, case["top_k"], *w, *rates, max_tokens, d_ff_shared=Hs, shared=shared)


def prepare(case, seed):
    rng = np.random.default_rng([int(seed) & 0xffffffff, 7])
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    T, M, E = case["tokens"], case["d_model"], case["n_experts"]
    s = State()
    for _ in range(case["layers"]):
        s.layers.append(_make_layer(case, rng))
    if case["layers"] > 1:
        s.stack = si.si_stack_create(s.layers)
    s.T, s.n_g = T, case["n_g"]
    s.x = torch.randn(T, M, generator=g, device="cuda").to(torch.bfloat16)
    s.logits = [None] * case["layers"]
    if case["router"] != "none":
        bias = torch.zeros(E)
        if case["router"] == "zipf":
            bias[torch.from_numpy(rng.permutation(E))] = -1.1 * torch.arange(1, E + 1, dtype=torch.float32).log()
        s.logits = [torch.randn(T, E, generator=g, device="cuda") + bias.cuda() for _ in range(case["layers"])]
    s.y = torch.empty(T, M, device="cuda", dtype=torch.float32)
    return s


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    ptr = [t.data_ptr() if t is not None else None for t in s.logits]
    if s.stack is not None:
        si.si_stack_forward(s.stack, s.x.data_ptr(), ptr, s.T, s.n_g, si.SI_AUTO, s.y.data_ptr(), stream=stream)
    else:
        si.si_layer_forward(s.layers[0], s.x.data_ptr(), ptr[0], s.T, s.n_g, si.SI_AUTO, s.y.data_ptr(), stream=stream)
    return s.y


# ------------------------------------------------------------------------------------------------ what a pass needs
def _experts_used(case):
    """Distinct routed experts of one call, averaged over a few draws of the router."""
    E, k, T = case["n_experts"], case["top_k"], case["tokens"]
    if E == 1:
        return 1.0
    rng = np.random.default_rng(3)
    bias = -1.1 * np.log(np.arange(1, E + 1)) if case["router"] == "zipf" else np.zeros(E)
    used = []
    for _ in range(16 if T <= 256 else 1):
        top = np.argpartition(-(rng.standard_normal((T, E)) + bias), k - 1, axis=1)[:, :k]
        used.append(np.unique(top).size)
    return float(np.mean(used))


def _weights(case, experts):
    return 3.0 * case["d_model"] * (experts * case["d_ff"] + case["d_ff_shared"])


def work(case):
    T, M = case["tokens"], case["d_model"]
    per_weight = 2.0 if case["dtype"] == "bf16" else 0.5 + 2.0 / GROUP
    layer = _weights(case, _experts_used(case)) * per_weight + T * M * (2 + 4) + (T * case["n_experts"] * 4 if case["router"] != "none" else 0)
    flops = 6.0 * T * M * (case["top_k"] * case["d_ff"] + case["d_ff_shared"])
    return {"bytes": layer * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    """About four times what each path was measured to be off from the same layer in 64 bits.

    Calls of few tokens keep the activations in fp32 and sum exact products in fp32 (measured: rel 8e-7, max 3e-6 with
    bf16 weights, 1.7e-6 and 8e-6 with 4-bit ones); the host's share of a split layer splits fp32 activations into two
    bf16 parts (max 2e-5).  Calls on the matrix cores round the activations to bf16 once (rel 1.7e-3, max 9.5e-3),
    with 4-bit weights those too (rel 2.8e-3, max 1.4e-2).  A stack rounds the hidden state to bf16 between layers,
    where two correct sums of a few elements fall on different sides of a rounding boundary, one bf16 step apart."""
    q4 = case["dtype"] == "q4"
    rows = -(-case["tokens"] * case["top_k"] // case["n_experts"])
    if not (case["tokens"] <= si.SI_DECODE_AUTO_T and rows <= si.SI_DECODE_AUTO_ROWS):
        return {"rel": 1.1e-2, "max": 6e-2} if q4 else {"rel": 7e-3, "max": 4e-2}
    if case["layers"] > 1:
        return {"rel": 4e-4, "max": 2e-2}
    if case["r_cc"] > 0:
        return {"rel": 4e-5, "max": 2e-4}
    return {"rel": 1e-5, "max": 5e-5}
