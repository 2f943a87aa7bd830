"""CPU tests of what the library's host side enqueues and in which order: the library runs in a child process against
stand-ins for the HIP runtime (hip_calls.c) that write its launches, event records and event waits down and run no kernel.
A layer call's statistics never arrive there, so it ends in an error after its launches; rank calls run to their end."""
import ctypes as C
import json
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EINVAL = -1
A, B = 0xA0000, 0xB0000                                  # two caller's streams


# ------------------------------------------------------------------------------------------ the child process
class Host:
    """The library behind the stand-ins; every tensor is an address that nobody reads."""

    def __init__(self, stub, T=4096, E=64, k=6, D=8, H=256, I=128):
        self.stub = C.CDLL(stub, mode=C.RTLD_GLOBAL)
        self.stub.calls_log.restype = C.c_char_p
        self.lib = C.CDLL(os.path.join(ROOT, "paper_2604_19503_amd", "librealb.so"))
        sys.path.insert(0, ROOT)
        from paper_2604_19503_amd import binding
        self.b = binding
        vp = C.c_void_p
        self.lib.realb_layer_forward.argtypes = [vp, vp, vp]
        self.lib.realb_rank_forward.argtypes = [vp, vp, C.c_int, vp]
        self.lib.realb_prefetch_join.argtypes = [vp, vp]
        self.lib.realb_combine.argtypes = [vp, vp, vp, vp, C.c_int, vp, vp]
        rows = [vp, C.c_int, vp, C.c_int, C.c_longlong]
        self.lib.realb_grouped_moe_ffn.argtypes = rows + [vp] * 10
        self.lib.realb_grouped_moe_ffn_gate_up.argtypes = rows + [vp] * 7
        self.lib.realb_grouped_moe_ffn_down.argtypes = rows + [vp] * 6
        self.cfg = binding.default_config(T, E, k, D, H, I)
        self.ctx = vp()
        assert self.lib.realb_create(C.byref(self.cfg), C.byref(self.ctx)) == 0
        self.addr = 0x10000000

    def new(self):
        self.addr += 0x100000
        return self.addr

    def io(self, overlap, force=-1, fp4=True, prefetch=False, T=None):
        io = self.b.LayerIO()
        for name, kind in io._fields_:
            if kind is C.c_void_p and not name.startswith("next_"):
                setattr(io, name, self.new())
        if not fp4:
            io.w13_q = io.w13_s = io.w2_q = io.w2_s = None
        if prefetch:
            for name in ("next_w13", "next_w2", "next_w13_q", "next_w13_s", "next_w2_q", "next_w2_s"):
                setattr(io, name, self.new())
        io.T = self.cfg.T_max if T is None else T
        io.rank, io.force, io.overlap = 0, force, overlap
        io.max_rows = io.T * min(self.cfg.k, self.cfg.E // self.cfg.D)
        return io

    def calls(self):
        """(return value, calls) of the last step: launches as ("launch", kernel, threads, stream), events as (what, event, stream)."""
        out = []
        for line in self.stub.calls_log().decode().splitlines():
            m = re.match(r"launch (\S+) grid (\d+) block (\d+) stream (\S+)", line)
            if m:
                out.append(["launch", m[1], int(m[2]) * int(m[3]), _num(m[4])])
            else:
                m = re.match(r"(record|wait) event (\S+) stream (\S+)", line)
                out.append([m[1], _num(m[2]), _num(m[3])])
        self.stub.calls_clear()
        return out

    def layer(self, io, stream):
        return self.lib.realb_layer_forward(self.ctx, C.byref(io), stream), self.calls()

    def rank(self, io, prec, stream):
        return self.lib.realb_rank_forward(self.ctx, C.byref(io), prec, stream), self.calls()

    def pending_prefetch(self, stream):
        """A rank call that leaves a prefetch pending; returns the event that marks its end."""
        io = self.io(0, prefetch=True)
        rc, calls = self.rank(io, 1, stream)
        assert rc == 0
        return [c for c in calls if c[0] == "record"][-1][1]


def _num(text):
    return 0 if text == "(nil)" else int(text, 16)


def refused_call(stub):
    """A refused call enqueues nothing and leaves a pending prefetch to the call that will consume it."""
    h = Host(stub)
    out = []
    for how in ("layer", "rank", "force"):
        ev = h.pending_prefetch(A)
        bad = h.io(4, force=7 if how == "force" else 1)
        if how != "force":
            bad.max_rows = 1
        rc, calls = h.rank(bad, 1, B) if how == "rank" else h.layer(bad, B)
        rc2, used = h.rank(h.io(4), 1, A)
        first = next(i for i, c in enumerate(used) if c[0] == "launch")
        out.append([rc, calls, rc2, ["wait", ev, A] in used[:first]])
    return out


def call_that_fails_behind_its_prefetch(stub):
    """Its own stream waits for the prefetch, so that the caller may free the buffers; nobody has to wait again."""
    h = Host(stub)
    h.stub.calls_fail(b"combine_kernel")
    rc, calls = h.rank(h.io(0, prefetch=True), 1, A)
    h.stub.calls_fail(b"")
    ev = [c for c in calls if c[0] == "record"][-1][1]
    rc2, used = h.rank(h.io(4), 1, A)
    return [rc, calls[-1] == ["wait", ev, A], rc2, [c for c in used if c[0] != "launch"]]


def encoding_behind_a_prefetch(stub):
    """Calls that encode their weights themselves while a prefetch is pending: (placement, precision call, waits for the prefetch
    before its first launch, the consuming call on another stream still waits); then the same under capture."""
    h = Host(stub)
    out = []
    for overlap in (0, 1, 3):
        for how in ("layer", "open", "rank"):
            for again in (False, True):                  # again: the call issues a prefetch of its own
                ev = h.pending_prefetch(A)
                io = h.io(overlap, force=-1 if how == "open" else 1, prefetch=again, T=4096)
                _, calls = h.rank(io, 1, A) if how == "rank" else h.layer(io, A)
                first = next(i for i, c in enumerate(calls) if c[0] == "launch")
                _, used = h.rank(h.io(4), 1, B)
                first_used = next(i for i, c in enumerate(used) if c[0] == "launch")
                out.append([overlap, how, again, ["wait", ev, A] in calls[:first], ["wait", ev, B] in used[:first_used]])
    ev = h.pending_prefetch(A)
    h.stub.calls_set_capturing(1)
    rc, calls = h.rank(h.io(1), 1, B)
    return out, [rc, [c for c in calls if c[0] != "launch"]]


def encoding_behind_an_ended_prefetch(stub):
    """The event waits of two layer calls that encode their own weights and of a consuming rank call on another stream, once
    the prefetch of a pipeline that nobody continued has ended."""
    h = Host(stub)
    h.pending_prefetch(A)
    h.stub.calls_set_events_done(1)
    calls = [h.layer(h.io(1, force=1), A)[1], h.layer(h.io(3, force=1), A)[1], h.rank(h.io(4), 1, B)[1]]
    return [[e for e in c if e[0] == "wait"] for c in calls]


def speculation_without_buffers(stub):
    h = Host(stub)
    out = []
    for T in (64, 4096):                                 # gate closed: the decision will be BF16; open
        rc, calls = h.layer(h.io(3, force=-1, fp4=False, T=T), A)
        out.append([rc, calls])
    forced = h.layer(h.io(3, force=0, fp4=False), A)     # forced BF16: nothing is speculated on
    plain = h.layer(h.io(1, force=-1, fp4=False), A)
    return out, [len([c for c in calls if c[0] == "launch"]) for _, calls in (forced, plain)]


def gemm_operands(stub):
    """(entry point, kernel selector, precision, with scale tensors) -> the launches' kernels and operands (activations, their scales,
    weights, their scales, output, its scales)."""
    h = Host(stub)
    offs, x, x_s, w13, w13_s, w2, w2_s, h_mid, h_s, y = (h.new() for _ in range(10))
    out = []
    for tile in (0, 2, 8, 16):
        h.lib.realb_set_gemm_tile(tile)
        for prec in (0, 1):
            for scales in (True, False) if prec == 0 else (True,):
                s = lambda t: t if scales else None
                calls = {"": (x, s(x_s), w13, s(w13_s), w2, s(w2_s), h_mid, s(h_s), y, A),
                         "_gate_up": (x, s(x_s), w13, s(w13_s), h_mid, s(h_s), A),
                         "_down": (h_mid, s(h_s), w2, s(w2_s), y, A)}
                for name, args in calls.items():
                    h.stub.calls_clear()
                    assert getattr(h.lib, "realb_grouped_moe_ffn" + name)(h.ctx, prec, offs, 8, 4096, *args) == 0
                    lines = h.stub.calls_log().decode().splitlines()
                    out.append([name, tile, prec, scales, [[l.split()[1], [_num(o) for o in l.split("operands ")[1].split()]] for l in lines]])
    return [x_s, w13_s, w2_s, h_s], out


def largest_grids(stub, T, H, force):
    """(return value, threads of the largest launch) of a rank call (force) or of combine alone (None)."""
    h = Host(stub, T=T, E=2, k=1, D=2, H=H)
    if force is None:
        rc, calls = h.lib.realb_combine(h.ctx, h.new(), h.new(), h.new(), T, h.new(), A), h.calls()
    else:
        rc, calls = h.rank(h.io(0), force, A)
    return rc, max(c[2] for c in calls if c[0] == "launch")


# ------------------------------------------------------------------------------------------ the tests
@pytest.fixture(scope="session")
def stub(tmp_path_factory):
    path = str(tmp_path_factory.mktemp("hip_calls") / "libhip_calls.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", path, os.path.join(ROOT, "tests", "hip_calls.c")], check=True)
    return path


def _run(stub, what, *args):
    res = subprocess.run([sys.executable, os.path.abspath(__file__), stub, what, json.dumps(args)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]
    return json.loads(res.stdout.splitlines()[-1])


def test_refused_call_leaves_a_pending_prefetch_alone(stub):
    """The refused call is on another stream than the pipeline's: were the prefetch marked as waited for there, the consuming
    call would read half-encoded weights."""
    for rc, enqueued, rc2, waits in _run(stub, "refused_call"):
        assert rc == EINVAL and enqueued == []
        assert rc2 == 0 and waits


def test_call_that_fails_behind_its_prefetch_waits_for_it(stub):
    rc, waited, rc2, events = _run(stub, "call_that_fails_behind_its_prefetch")
    assert rc < 0 and waited
    assert rc2 == 0 and events == []


def test_call_that_encodes_its_weights_waits_for_a_pending_prefetch(stub):
    """The prefetch may be writing the very buffers that the call encodes into.  Only the call that consumes it (or issues the
    next one) takes it off the list; an encoding call recorded into a graph, where an event from outside cannot be waited
    for, is recorded as before."""
    eager, (rc, captured) = _run(stub, "encoding_behind_a_prefetch")
    for overlap, how, again, waits, still_pending in eager:
        assert waits, (overlap, how, again)
        # (a layer call ends in an error here before it gets to its own prefetch; a rank call has replaced the pending one)
        assert still_pending or again, (overlap, how, again)
    assert rc == 0 and captured == []


def test_an_ended_prefetch_is_waited_for_no_more(stub):
    """A wait costs the stream microseconds also for an event that has completed."""
    assert _run(stub, "encoding_behind_an_ended_prefetch") == [[], [], []]


def test_speculative_encoding_needs_its_buffers(stub):
    """Without the FP4 weight buffers a speculative call is refused before anything is enqueued, whatever the decision would be."""
    refused, launches = _run(stub, "speculation_without_buffers")
    assert refused == [[EINVAL, []], [EINVAL, []]]
    assert all(n > 0 for n in launches)


def test_bf16_gemms_get_no_scale_tensors(stub):
    """BF16 ignores the scale pointers: its kernels get the same operands whether a caller passes any or not (a kernel that took a
    pointer to scales for the sign of FP4 would follow FP4's rules in BF16).  FP4's kernels get them all."""
    scales, launches = _run(stub, "gemm_operands")
    bf16 = {(name, tile, with_scales): l for name, tile, prec, with_scales, l in launches if prec == 0}
    for name, tile, with_scales in bf16:
        assert bf16[name, tile, with_scales] and bf16[name, tile, with_scales] == bf16[name, tile, False], (name, tile)
        assert not any(o in scales for _, ops in bf16[name, tile, with_scales] for o in ops), (name, tile)
    x_s, w13_s, w2_s, h_s = scales
    for name, tile, prec, _, l in launches:
        if prec == 1:
            want = {"": [[x_s, w13_s, h_s], [h_s, w2_s, 0]], "_gate_up": [[x_s, w13_s, h_s]], "_down": [[h_s, w2_s, 0]]}[name]
            assert [[ops[1], ops[3], ops[5]] for _, ops in l] == want, (name, tile)


@pytest.mark.parametrize("T,H,force", [
    ((1 << 22) + 3, 8192, None),                         # combine: 16 panels per token
    ((1 << 26) + 5, 128, 0),                             # rows that the gate/up GEMM cannot fetch itself
    ((1 << 26) - 1, 128, 1),                             # FP4, tokens encoded beside the ranking kernel
])
def test_no_launch_passes_the_runtimes_grid_limit(stub, T, H, force):
    """Fewer than 2^32 threads in a launch, at sizes that a context is created for."""
    rc, threads = _run(stub, "largest_grids", T, H, force)
    assert rc == 0 and threads < 1 << 32


if __name__ == "__main__":
    print(json.dumps(globals()[sys.argv[2]](sys.argv[1], *json.loads(sys.argv[3]))))
