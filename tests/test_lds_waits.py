"""The 4-bit prompt-phase GEMMs write converted weights to LDS by inline assembly, which the compiler does not wait for, and pass barriers
without the memory fence of __syncthreads().  The next body of a block (another tile, or the second pass over one) lays its rings out
differently, so a store still on its way when a main loop ends may land in what another wave has loaded for the next body.  Read
from the built kernels' own code: on every path from an LDS store out of its innermost loop, before any direct load to LDS, the
wave waits for its LDS operations (lgkmcnt(0)) and then passes a barrier."""
import os
import re
import subprocess

import paper_2411_15715_amd.build as lib_build

LLVM = os.environ.get("SI_LLVM_BIN", "/opt/rocm/lib/llvm/bin")
KERNELS = ["k_prefill_gateup_q4", "k_prefill_down_q4"]


def _kernels(tmp_path):
    """name -> [(address, instruction, branch target or None)] of the device code in the object file of prefill.hip"""
    obj = os.path.join(lib_build.OBJ, "prefill.hip.o")
    if not os.path.exists(obj):
        lib_build.build(force=False)
    local = tmp_path / "prefill.o"
    local.write_bytes(open(obj, "rb").read())
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", local.name], cwd=tmp_path, check=True, capture_output=True)
    code = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    assert len(code) == 1, code
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", code[0]], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
    out, name, base = {}, None, 0
    for line in text.splitlines():
        m = re.match(r"([0-9a-f]+) <(.+)>:$", line)
        if m:
            name, base = m.group(2), int(m.group(1), 16)
            out[name] = []
            continue
        m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if not m or name is None:
            continue
        t = re.search(r"<%s(?:\+0x([0-9a-f]+))?>$" % re.escape(name), line)
        out[name].append((int(m.group(2), 16), m.group(1), base + int(t.group(1) or "0", 16) if t else None))
    return out


def _blocks(code):
    """basic blocks: list of (first, last + 1) instruction, successors of each"""
    index = {a: i for i, (a, _, _) in enumerate(code)}
    cuts = {0, len(code)}
    for i, (_, op, target) in enumerate(code):
        assert not op.startswith(("s_setpc", "s_swappc")), op
        if op.startswith(("s_branch", "s_cbranch", "s_endpgm")):
            cuts.add(i + 1)
            if target is not None:
                cuts.add(index[target])
    cuts = sorted(cuts)
    blocks = list(zip(cuts, cuts[1:]))
    start = {b[0]: n for n, b in enumerate(blocks)}
    succ = []
    for n, (_, end) in enumerate(blocks):
        _, op, target = code[end - 1]
        branch = op.startswith(("s_branch", "s_cbranch"))
        assert not branch or target is not None, op
        nxt = [start[index[target]]] if branch else []
        if not op.startswith(("s_branch", "s_endpgm")) and n + 1 < len(blocks):
            nxt.append(n + 1)
        succ.append(nxt)
    return blocks, succ


def _reach(n, succ, inside):
    seen, todo = set(), [n]
    while todo:
        for m in succ[todo.pop()]:
            if m in inside and m not in seen:
                seen.add(m)
                todo.append(m)
    return seen


def _innermost_loop(n, succ):
    """blocks of the innermost loop around block n (empty: none): of the blocks on a cycle through n, the headers (entered from outside)
    are taken out until no cycle is left"""
    pred = [[] for _ in succ]
    for a, nxt in enumerate(succ):
        for b in nxt:
            pred[b].append(a)
    inside, loop = set(range(len(succ))), set()
    while True:
        cycle = _reach(n, succ, inside) & _reach(n, pred, inside)
        if n not in cycle:
            return loop
        loop = cycle
        heads = {b for b in cycle if any(a not in cycle for a in pred[b])}
        if n in heads or not heads:
            return loop
        inside = cycle - heads


def _overtaken(code):
    """number of LDS stores inside a main loop (one with matrix instructions), and (store, load) addresses where a direct load to LDS
    outside the loop may overtake one of them"""
    blocks, succ = _blocks(code)
    n_stores, bad = 0, None
    for n, (b0, b1) in enumerate(blocks):
        stores = [i for i in range(b0, b1) if code[i][1].startswith("ds_write_b128")]
        loop = _innermost_loop(n, succ) if stores else set()
        if not any(code[i][1].startswith("v_mfma") for b in loop for i in range(*blocks[b])):
            continue
        n_stores += len(stores)
        # from the last store of the block on: (block, first instruction, waited for)
        seen, todo = set(), [(n, stores[-1] + 1, False)]
        while todo:
            b, first, waited = todo.pop()
            if (b, first, waited) in seen:
                continue
            seen.add((b, first, waited))
            done = False
            for i in range(first, blocks[b][1]):
                a, op, _ = code[i]
                waited = waited or (op.startswith("s_waitcnt") and "lgkmcnt(0)" in op)
                if waited and op.startswith("s_barrier"):
                    done = True
                    break
                if op.startswith("global_load_lds") and b not in loop:
                    bad = bad or (hex(code[stores[-1]][0]), hex(a))
            if not done:
                todo += [(m, blocks[m][0], waited) for m in succ[b]]
    return n_stores, bad


def test_converted_weights_have_landed_when_a_loop_ends(tmp_path):
    kernels = _kernels(tmp_path)
    for short in KERNELS:
        names = [n for n in kernels if re.search(r"\d%s(?:I|E)" % short, n)]
        assert names, short
        for name in names:
            n_stores, bad = _overtaken(kernels[name])
            assert n_stores >= 8 * 4, name  # (eight bodies, four pieces of a tile each)
            assert bad is None, "%s: the LDS store at %s may be overtaken by the load at %s" % ((short,) + bad)
