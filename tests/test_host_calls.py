"""The library's host logic on a stand-in for the HIP runtime (hip_stub.c: device memory is host memory, kernels are not run): which
allocations, copies and launches a call makes, and what is left of a layer after a call that fails half-way.  Each test runs in
a process of its own, which loads the stand-in before the library."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROLOGUE = """
import ctypes, sys
sys.path.insert(0, %r)
stub = ctypes.CDLL(%r, mode=ctypes.RTLD_GLOBAL)
stub.hip_stub_log.restype = ctypes.c_char_p
import numpy as np
import paper_2411_15715_amd as si

def log():
    out = stub.hip_stub_log().decode().splitlines()
    stub.hip_stub_clear()
    return out

def calls(lines, *names):
    return [l for l in lines if l.split()[0] in names]

def layer(M, H, split, E=1, k=1, Hs=0, max_tokens=64, **kw):
    w = [np.zeros((E, H, M), np.uint16) for _ in range(3)]
    s = tuple(np.zeros((Hs, M), np.uint16) for _ in range(3)) if Hs else None
    return si.si_layer_create(M, H, E, k, *w, *split, max_tokens, d_ff_shared=Hs, shared=s, **kw)

def forward(h, M, T, E=1, n_g=0, mode=si.SI_AUTO):
    x, y, lg = np.zeros((T, M), np.uint16), np.zeros((T, M), np.float32), np.zeros((T, E), np.float32)
    stub.hip_stub_rows(T, T - n_g)
    si.si_layer_forward(h, x.ctypes.data, lg.ctypes.data if E > 1 else None, T, n_g, mode, y.ctypes.data, stream=0)

def attempt(f, *a, **kw):
    try:
        f(*a, **kw)
        return si.SI_OK
    except si.ScheInferError as e:
        return e.code
"""


@pytest.fixture(scope="session")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("hip_stub")
    so = str(d / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-fPIC", "-shared", "-Wall", "-Wextra", "-Werror", "-o", so, os.path.join(ROOT, "tests", "hip_stub.c")], check=True)

    def run(script):
        r = subprocess.run([sys.executable, "-c", PROLOGUE % (ROOT, so) + textwrap.dedent(script)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, "exit code %d\n%s\n%s" % (r.returncode, r.stdout[-2000:], r.stderr[-4000:])
        return r.stdout

    return run


@pytest.mark.parametrize("call", ["hipMalloc", "hipHostMalloc", "hipEventCreateWithFlags"])
def test_resplit_that_runs_out_of_memory_leaves_a_whole_layer(host, call):
    """Every allocation of a re-slicing that gives a resident layer its first host parts fails once.  Calls on the layer then either work
    or are refused, and the same re-slicing works when it is tried again; no copy or launch ever names a null buffer."""
    out = host("""
    def run(h):
        codes = [attempt(forward, h, 256, 4, n_g=n_g, mode=mode) for mode in (si.SI_DECODE, si.SI_PREFILL) for n_g in (0, 4)]
        lines = log()
        copies = calls(lines, "k_copy_piece", "hipMemcpyAsync")
        assert not any("(nil) ->" in l or "-> (nil)" in l for l in copies), copies
        return codes, copies

    n_failed = 0
    for nth in range(1, 12):
        h = layer(256, 704, (1.0, 0.0, 0.0))
        stub.hip_stub_fail(b"%s", nth)
        rc = attempt(si.si_layer_resplit, h, 0.4, 0.3, 0.3)
        stub.hip_stub_fail(b"", 0)
        n_failed += rc != si.SI_OK
        if rc != si.SI_OK:
            assert rc in (si.SI_ENOMEM, si.SI_EHIP), rc
            resident = si.si_layer_split_info(h)["n_gg"] == 704
            codes, _ = run(h)
            assert codes == [si.SI_OK if resident else si.SI_EHIP] * 4, (nth, codes)
            si.si_layer_resplit(h, 0.4, 0.3, 0.3)
        codes, copies = run(h)
        assert codes == [si.SI_OK] * 4 and copies, (codes, copies)
        si.si_layer_destroy(h)
    print(n_failed)
    """ % call)
    assert int(out) >= 1


def test_prefetch_to_a_layer_without_staging_buffers(host):
    """A stack whose second layer ran out of memory while it was re-sliced: the first layer's call does not copy ahead for it, the
    second's is refused."""
    host("""
    a, b = layer(256, 704, (0.4, 0.6, 0.0)), layer(256, 704, (1.0, 0.0, 0.0))
    stub.hip_stub_fail(b"hipMalloc", 3)
    assert attempt(si.si_layer_resplit, b, 0.4, 0.6, 0.0) == si.SI_ENOMEM
    S = si.si_stack_create([a, b])
    x, y = np.zeros((4, 256), np.uint16), np.zeros((4, 256), np.float32)
    log()
    args = (S, x.ctypes.data, None, 4, 0, si.SI_AUTO, y.ctypes.data)
    assert attempt(si.si_stack_forward, *args, prefetch=1, stream=0) == si.SI_EHIP
    assert not any("(nil) ->" in l or "-> (nil)" in l for l in log())
    si.si_layer_resplit(b, 0.4, 0.6, 0.0)
    si.si_stack_forward(*args, prefetch=1, stream=0)
    """)


@pytest.mark.parametrize("failing", ["k_prefill_down", "k_prefill_combine"])
def test_tile_queues_after_a_call_that_failed(host, failing):
    """A prompt call that ends between FC1 and its merge leaves the tile counters as FC1 or FC2 left them: the next call clears them
    before its FC1 launch, once; a decode call in between does not."""
    host("""
    h = layer(256, 704, (1.0, 0.0, 0.0))
    def prompt():
        stub.hip_stub_clear()
        rc = attempt(forward, h, 256, 64, mode=si.SI_PREFILL)
        return rc, [l.split()[0] for l in calls(log(), "k_fill_zero", "k_prefill_gateup", "k_prefill_down", "k_prefill_combine")]
    usual = (si.SI_OK, ["k_prefill_gateup", "k_prefill_down", "k_prefill_combine"])
    prompt()
    assert prompt() == usual
    stub.hip_stub_fail(b"%s", 1)
    assert prompt()[0] == si.SI_EHIP
    forward(h, 256, 4)
    assert prompt() == (si.SI_OK, ["k_fill_zero"] + usual[1])
    assert prompt() == usual
    """ % failing)


@pytest.mark.parametrize("kw", [dict(), dict(E=4, k=2), dict(E=4, k=2, Hs=256)])
def test_a_recorded_prompt_call_clears_its_tile_queues(host, kw):
    """A graph may be replayed after a call that failed, which no host flag tells it: every recorded prompt call clears the counters
    itself, before FC1, whatever state the layer is in, and leaves what the host knows of them alone."""
    host("""
    kw = %r
    h = layer(256, 704, (1.0, 0.0, 0.0), **kw)
    def prompt(capturing):
        stub.hip_stub_clear()
        stub.hip_stub_capturing(capturing)
        rc = attempt(forward, h, 256, 64, E=kw.get("E", 1), mode=si.SI_PREFILL)
        stub.hip_stub_capturing(0)
        names = [l.split()[0] for l in calls(log(), "k_fill_zero", "k_prefill_gateup")]
        assert names[-1] == "k_prefill_gateup" or rc
        return rc, len(names) - 1
    prompt(0)
    assert prompt(0) == (si.SI_OK, 0)
    assert prompt(1) == (si.SI_OK, 1)
    assert prompt(1) == (si.SI_OK, 1)
    assert prompt(0) == (si.SI_OK, 0)
    stub.hip_stub_fail(b"k_prefill_down", 1)
    prompt(0)
    assert prompt(1) == (si.SI_OK, 1)
    assert prompt(0) == (si.SI_OK, 1)
    assert prompt(0) == (si.SI_OK, 0)
    """ % kw)


def test_which_parts_a_kernel_copies(host):
    """Generation calls whose streamed part is not read in place (test_which_parts_are_read_in_place): a dense layer's parts of up to 32 MB where
    the host computes a share, of up to 8 MB without, of several experts 4 MB, both with few rows, each whole whatever the size of a staging
    buffer.  All else uses the ring, in pieces: larger parts to their last piece, many rows, calls beside a large resident part.  Chunks of 64 columns of
    d_model 4096 are 1.5 MB."""
    host("""
    def run(M, chunks, cg, cc=0, stage_mib=0, T=1, E=1, k=1, Hs=0, n_g=0, n_stage=0, mode=si.SI_DECODE):
        split = ((chunks - cg - cc) / chunks, cg / chunks, cc / chunks)
        h = layer(M, 64 * chunks, split, E=E, k=k, Hs=Hs, stage_mib=stage_mib, n_stage=n_stage)
        log()
        forward(h, M, T, E=E, n_g=n_g, mode=mode)
        lines = log()
        si.si_layer_destroy(h)
        return len(calls(lines, "k_copy_piece")), len(calls(lines, "hipMemcpyAsync"))
    # dense, a host part
    assert run(4096, 24, 21, 1) == (1, 0)                       # 31.5 MB
    assert run(4096, 24, 21, 1, stage_mib=16) == (1, 0)         # ... in one piece
    assert run(4096, 24, 22, 1) == (0, 1)                       # 33 MB
    assert run(4096, 24, 22, 1, stage_mib=16) == (0, 3)         # ... pieces of 10, 10 and 2 chunks
    assert run(4096, 64, 61, 1, stage_mib=16, n_stage=4) == (0, 8)  # whole slots of 8 chunks
    assert run(4096, 24, 10, 10, T=4, n_g=2) == (2, 0)          # CG and CG'
    assert run(4096, 48, 1, 1) == (0, 1)                        # resident part of 69 MB
    assert run(4096, 24, 21, 1, mode=si.SI_PREFILL) == (0, 1)
    # dense without a host share, and several experts (every one has T rows here): by the part's size, by rows x d_model
    assert run(4096, 24, 2) == (1, 0)                           # 3 MB
    assert run(4096, 24, 5) == (1, 0)                           # 7.5 MB
    assert run(4096, 24, 6) == (0, 1)                           # 9 MB
    assert run(4096, 24, 2, T=2) == (0, 1)
    assert run(4096, 24, 2, 2, T=1, n_g=1) == (2, 0)            # CG' takes the host's share
    assert run(4096, 24, 6, 2, T=1, n_g=1) == (1, 1)
    assert run(4096, 8, 2, E=8, k=2, stage_mib=1) == (8, 0)
    assert run(4096, 8, 3, E=8, k=2) == (0, 8)
    assert run(4096, 8, 2, E=8, k=2, T=2) == (0, 8)
    assert run(1024, 8, 2, E=8, k=2, T=6) == (8, 0)
    assert run(1024, 8, 2, E=8, k=2, T=7) == (0, 8)
    assert run(1024, 8, 2, 2, E=8, k=2, T=7, n_g=1) == (8, 8)   # CG of 7 rows, CG' of 1
    assert run(8192, 8, 1, E=8, k=2) == (0, 8)
    assert run(1024, 8, 2, E=1, Hs=512) == (2, 0)
    """)


def test_which_parts_are_read_in_place(host):
    """Generation calls of up to four tokens: a bf16 dense layer's streamed part of up to 8 MB where the host computes a share, of up to 2 MB
    without, beside a resident part of up to 64 MB, takes no copy and no launch of its own, recorded or not.  Not with CG' rows, in a stack, while the
    call is timed, on the prompt path, for 4-bit weights or beside other experts.  Chunks are 96 KiB at d_model 256, 384 KiB at 1024, 768 KiB at 2048."""
    host("""
    def calls_of(h, f):
        log()
        f()
        lines = log()
        n = lambda *names: len(calls(lines, *names))
        return n("k_copy_piece", "hipMemcpyAsync"), n("k_decode_gateup", "k_decode_gateup_q4"), n("k_decode_down", "k_decode_down_q4"), n("hipStreamWaitEvent")

    def run(M, chunks, cg, cc=0, T=1, n_g=0, mode=si.SI_DECODE, timed=0, E=1, Hs=0):
        h = layer(M, 64 * chunks, ((chunks - cg - cc) / chunks, cg / chunks, cc / chunks), E=E, Hs=Hs)
        si.si_layer_set_profiling(h, timed)
        out = calls_of(h, lambda: forward(h, M, T, E=E, n_g=n_g, mode=mode))
        st = si.si_layer_stats(h)
        if cg and not n_g and E == 1 and not Hs:
            assert st["n_copies"] == 1 and st["bytes_streamed"] == cg * 384 * M, st  # one streamed piece, however it travels
        si.si_layer_destroy(h)
        return out
    IN_PLACE = (0, 1, 1, 0)
    copied = lambda out: out[:3] == (1, 2, 2)
    for T in (1, 2, 3, 4):
        assert run(256, 11, 3, 3, T=T) == IN_PLACE
        assert run(256, 40, 21, T=T) == IN_PLACE            # 1.97 MB
        assert copied(run(256, 40, 22, T=T))                # 2.06 MB
        assert run(2048, 24, 10, 1, T=T) == IN_PLACE        # 7.5 MB and a host share
        assert copied(run(2048, 24, 11, 1, T=T))            # 8.25 MB
    assert copied(run(256, 11, 3, 3, T=5)) and copied(run(256, 40, 21, T=5))
    assert run(1024, 170, 1, 1) == IN_PLACE                 # beside 63 MB
    assert copied(run(1024, 173, 1, 1))                     # beside 64.1 MB
    assert copied(run(256, 11, 3, 3, T=4, timed=1)) and copied(run(256, 40, 21, timed=1))
    assert run(256, 11, 3, 3, T=4, n_g=2)[:3] == (2, 3, 3)  # CG and CG'
    assert run(256, 11, 8, 3)[:2] == (1, 1)                 # nothing resident to share launches with
    assert run(256, 11, 3, 3, T=4, mode=si.SI_PREFILL)[0] == 1
    assert run(256, 11, 3, 0, E=4)[0] == 4
    assert run(256, 11, 3, 0, Hs=704)[0] == 2
    h = layer(256, 704, (8 / 11, 3 / 11, 0.0))
    for capturing in (1, 0):
        stub.hip_stub_capturing(capturing)
        assert calls_of(h, lambda: forward(h, 256, 4, mode=si.SI_DECODE)) == IN_PLACE
    x, y = np.zeros((4, 256), np.uint16), np.zeros((4, 256), np.float32)
    S = si.si_stack_create([h])
    assert copied(calls_of(h, lambda: si.si_stack_forward(S, x.ctypes.data, None, 4, 0, si.SI_DECODE, y.ctypes.data, prefetch=0, stream=0)))
    si.si_stack_destroy(S)
    assert calls_of(h, lambda: forward(h, 256, 4, mode=si.SI_DECODE)) == IN_PLACE
    w = {"q_gate": np.zeros((1, 704, 128), np.uint8), "q_up": np.zeros((1, 704, 128), np.uint8), "q_down": np.zeros((1, 704, 128), np.uint8),
         "z_gate": np.zeros((1, 704, 4), np.uint16), "z_up": np.zeros((1, 704, 4), np.uint16), "z_down": np.zeros((1, 11, 256), np.uint16)}
    h = si.si_layer_create_q4(256, 704, 1, 1, w, 8 / 11, 3 / 11, 0.0, 8)
    assert copied(calls_of(h, lambda: forward(h, 256, 4, mode=si.SI_DECODE)))
    """)


def test_the_buffer_of_direct_copies_is_allocated_where_it_can_be_used(host):
    host("""
    def sizes(M, chunks, cg, cc=0, stage_mib=64, E=1, k=1):
        log()
        h = layer(M, 64 * chunks, ((chunks - cg - cc) / chunks, cg / chunks, cc / chunks), E=E, k=k, stage_mib=stage_mib)
        used = [int(l.split()[1]) // (384 * M) for l in calls(log(), "hipMalloc")]  # in chunks
        ring = max(8, (stage_mib << 20) // (384 * M))
        at = used.index(ring, 0 if chunks == cg + cc else 1)
        assert used[at:at + 2] == [ring] * 2, used
        return h, used[at + 2]
    assert sizes(4096, 24, 9, 11)[1] == 11           # the larger part
    assert sizes(4096, 24, 10)[1] == 10              # nothing on the host: a recorded call
    assert sizes(4096, 64, 60, stage_mib=16)[1] == 10  # ... in pieces
    assert sizes(4096, 64, 30, 31)[1] == 0           # more than 32 MB
    assert sizes(4096, 48, 1, 1)[1] == 0             # beside 69 MB
    assert sizes(4096, 8, 2, E=8, k=2)[1] == 2
    assert sizes(4096, 8, 3, E=8, k=2)[1] == 0       # more than 4 MB
    assert sizes(8192, 8, 1, E=8, k=2)[1] == 0       # one row is too many
    # no memory for it: the layer streams through the ring, and a later re-slicing tries again
    stub.hip_stub_fail(b"hipMalloc", 4)
    h = layer(4096, 64 * 24, (4 / 24, 9 / 24, 11 / 24), stage_mib=1)
    log()
    forward(h, 4096, 1)
    lines = log()
    assert not calls(lines, "k_copy_piece") and len(calls(lines, "hipMemcpyAsync")) == 2, lines  # (pieces of 8 chunks at most)
    si.si_layer_resplit(h, 6 / 24, 7 / 24, 11 / 24)
    log()
    forward(h, 4096, 1)
    copies = calls(log(), "k_copy_piece", "hipMemcpyAsync")
    assert len(copies) == 1 and copies[0].startswith("k_copy_piece") and "(nil)" not in copies[0].split(" on ")[0], copies
    """)


@pytest.mark.parametrize("dense", [True, False])
def test_pieces_copied_ahead_stay_in_the_ring(host, dense):
    """A part whose first pieces were copied ahead after the layer before comes from the ring altogether, though it is small."""
    host("""
    kw = dict(stage_mib=1) if %r else dict(E=4, k=2, Hs=960)
    E = kw.get("E", 1)
    layers = [layer(256, 960, (2 / 15, 12 / 15, 1 / 15), **kw) for _ in range(2)]
    S = si.si_stack_create(layers)
    x, y, lg = np.zeros((4, 256), np.uint16), np.zeros((4, 256), np.float32), np.zeros((4, 4), np.float32)
    stub.hip_stub_rows(4, 4)
    per_call = []
    for prefetch in (0, 1):
        log()
        si.si_stack_forward(S, x.ctypes.data, [lg.ctypes.data] * 2 if E > 1 else None, 4, 0, si.SI_DECODE, y.ctypes.data, prefetch=prefetch, stream=0)
        lines = log()
        per_call.append((len(calls(lines, "k_copy_piece")), len(calls(lines, "hipMemcpyAsync"))))
    n = E if E > 1 else 0
    # 12 chunks of 96 KB; ring pieces of 10 chunks (1 MiB) or all
    assert per_call[0] == (2 * (n + 1), 0), per_call
    assert per_call[1] == (2 * n + 1, 2 if E == 1 else 1), per_call
    """ % dense)


def test_recorded_calls_stay_off_the_copy_stream(host):
    """A generation call of a dense layer without a host share can be recorded while its pieces fit the kernel's buffer, whatever its
    rows: nothing of it is on the copy stream.  Larger pieces are not made to fit."""
    host("""
    def run(M, chunks, cg, T=1, stage_mib=0, n_g=0, cc=0):
        h = layer(M, 64 * chunks, ((chunks - cg - cc) / chunks, cg / chunks, cc / chunks), stage_mib=stage_mib)
        out = []
        for capturing in (0, 1, 0):
            stub.hip_stub_capturing(capturing)
            log()
            forward(h, M, T, n_g=n_g, mode=si.SI_DECODE)
            lines = log()
            stub.hip_stub_capturing(0)
            out.append((len(calls(lines, "k_copy_piece")), len(calls(lines, "hipMemcpyAsync")), len(calls(lines, "hipStreamWaitEvent"))))
        si.si_layer_destroy(h)
        assert out[0][:2] == out[2][:2], out
        return out[0][:2], out[1]
    assert run(1024, 16, 8, T=8) == ((0, 1), (1, 0, 0))
    assert run(4096, 24, 21, T=16) == ((0, 1), (1, 0, 0))
    assert run(4096, 64, 60, stage_mib=16) == ((0, 8), (8, 0, 0))
    assert run(4096, 24, 10, cc=10, T=2, n_g=2) == ((0, 2), (2, 0, 0))
    assert run(4096, 24, 22)[1][:2] == (0, 1)
    """)


def test_a_new_layer_has_its_tile_queues_cleared_by_its_first_prompt_call(host):
    """Creation does not touch the counters; the first prompt call clears them before FC1, generation calls before it do not."""
    host("""
    h = layer(256, 704, (1.0, 0.0, 0.0))
    assert not calls(log(), "hipMemset", "k_fill_zero")
    forward(h, 256, 4)
    assert not calls(log(), "hipMemset", "k_fill_zero")
    for n in (1, 0):
        forward(h, 256, 64, mode=si.SI_PREFILL)
        names = [l.split()[0] for l in calls(log(), "hipMemset", "k_fill_zero", "k_prefill_gateup")]
        assert names == ["k_fill_zero"] * n + ["k_prefill_gateup"], names
    """)


@pytest.mark.parametrize("M,H,split,kw", [(1024, 1920, (0.2, 0.6, 0.2), dict(stage_mib=1)), (256, 704, (0.4, 0.3, 0.3), dict(E=4, k=2, Hs=640)),
                                          (256, 704, (0.4, 0.6, 0.0), dict()), (256, 704, (1.0, 0.0, 0.0), dict(E=4, k=2))])
def test_a_call_after_one_that_failed_anywhere(host, M, H, split, kw):
    """Every copy, event and launch of a call fails once.  The call reports it, and the next one succeeds with the launches and copies of
    an undisturbed call (a prompt call with the clearing of the tile queues before them)."""
    out = host("""
    M, H, split, kw = %r, %r, %r, %r
    E = kw.get("E", 1)
    names = ["hipMemcpyAsync", "hipEventRecord", "hipStreamWaitEvent", "hipEventSynchronize", "k_copy_piece", "k_handoff", "k_decode_gateup", "k_decode_down",
             "k_decode_combine", "k_prefill_gateup", "k_prefill_down", "k_prefill_combine", "k_topk", "k_assign", "k_route_few", "k_route_small"]
    n = 0
    for mode, T, n_g in ((si.SI_DECODE, 4, 0), (si.SI_DECODE, 4, 2), (si.SI_PREFILL, 40, 0), (si.SI_PREFILL, 40, 20)):
        h = layer(M, H, split, **kw)
        def call():
            log()
            rc = attempt(forward, h, M, T, E=E, n_g=n_g, mode=mode)
            return rc, [l.split()[0] + " FAILED" * l.endswith("FAILED") for l in log()]
        for _ in range(3):
            rc, clean = call()
            assert rc == si.SI_OK, si.si_last_error()
        for name in names:
            for nth in range(1, clean.count(name) + 1):
                stub.hip_stub_fail(name.encode(), nth)
                rc, lines = call()
                assert rc == si.SI_EHIP and name + " FAILED" in lines, (mode, name, nth, rc)
                rc, lines = call()
                if mode == si.SI_PREFILL:
                    assert lines.count("k_fill_zero") == clean.count("k_fill_zero") + 1
                    lines.remove("k_fill_zero")
                assert rc == si.SI_OK and lines == clean, (mode, name, nth, rc, lines, clean)
                n += 1
        si.si_layer_destroy(h)
    print(n)
    """ % (M, H, split, kw))
    assert int(out) > 10


def test_the_gate_up_kernel_of_a_4bit_expert_does_not_follow_the_cut_of_its_parts(host):
    """The two 4-bit gate/up kernels sum a row in different orders: all launches over one expert's columns by itself take the same one,
    whatever the size of the part, of a staging buffer and of the pieces.  120 chunks of d_model 6720 are 82 MB."""
    host("""
    def layer_q4(M, H, split, E, k, Hs, stage_mib):
        w = {}
        for pre, lead, h in (("", (E,), H), ("s", (), Hs)):
            if h:
                for n in ("gate", "up", "down"):
                    w[pre + "q_" + n] = np.zeros(lead + (h, M // 2), np.uint8)
                w[pre + "z_gate"], w[pre + "z_up"] = (np.zeros(lead + (h, M // 64), np.uint16) for _ in range(2))
                w[pre + "z_down"] = np.zeros(lead + (h // 64, M), np.uint16)
        return si.si_layer_create_q4(M, H, E, k, w, *split, 16, d_ff_shared=Hs, stage_mib=stage_mib)

    def kernels(M, chunks, cg, cc=0, stage_mib=0, E=1, k=1, sh=0, T=2, n_g=0):
        h = layer_q4(M, 64 * chunks, ((chunks - cg - cc) / chunks, cg / chunks, cc / chunks), E, k, 64 * sh, stage_mib)
        log()
        forward(h, M, T, E=E, n_g=n_g, mode=si.SI_DECODE)
        names = [l.split()[0] for l in log() if l.startswith("k_decode_gateup")]
        si.si_layer_destroy(h)
        return set(names), len(names)

    WHOLE, SPLIT = "k_decode_gateup_q4", "k_decode_gateup_q4_split"
    # one launch or many: whole parts, pieces of 23 chunks, parts on both sides of 96 and of 128 chunks
    for M, chunks, want in ((6720, 120, WHOLE), (6720, 140, SPLIT), (6720, 96, SPLIT), (8192, 120, SPLIT), (6592, 96, WHOLE)):
        assert kernels(M, chunks, 0)[0] == {want}
        for cg, cc, n_g in ((chunks, 0, 0), (chunks - 20, 0, 0), (chunks // 3, 0, 0), (chunks // 3, chunks // 3, 2)):
            for stage_mib in (0, 16):
                names, n = kernels(M, chunks, cg, cc, stage_mib, n_g=n_g)
                assert names == {want} and (n > 2 or not stage_mib), (M, chunks, cg, stage_mib, names, n)
    # the streamed experts of several, and a shared expert by itself
    for stage_mib in (0, 16):
        assert kernels(6720, 110, 110, stage_mib=stage_mib, E=2)[0] == {WHOLE}
        assert kernels(6720, 24, 24, stage_mib=stage_mib, E=2, sh=110)[0] == {SPLIT, WHOLE}
        assert kernels(6720, 24, 24, stage_mib=stage_mib, E=2, sh=48)[0] == {SPLIT}
    """)
