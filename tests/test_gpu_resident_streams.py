"""The resident sweep as one of several users of the device: a caller's own
graph capture, operators on streams of their own."""
import sys

import numpy as np
import pytest

from paper_2006_16861_amd import inputs

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


def host(t):
    return t.detach().cpu().numpy()


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / max(np.linalg.norm(b.ravel()), 1e-300))


def note(msg):
    print(f"[case] {msg}", file=sys.stderr, flush=True)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
def test_callers_capture_after_a_warm_up(prec, variant):
    """With use_graph = 0 a caller may capture the application after one eager
    call: it takes the blocked sweep on fields that the eager call allocated.
    Replays on changed inputs, with eager work between them, are bit for bit
    what that sweep gives eagerly."""
    import torch
    from paper_2006_16861_amd import tdp
    note(f"capture after a warm-up, prec {prec} variant {variant}")
    p = inputs.random_medium((150, 140), seed=71, width=4)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g, ref = (tdp.operator_from_problem(p, prec=prec) for _ in range(2))
        g.set_tuning(use_graph=0)
        ref.set_tuning(kernel=2, tb_depth=8, tile=8 if prec else 5)
        F = dev(p.F)
        out = torch.empty_like(F)
        g.precond(F, 2, 0.25, out=out, variant=variant)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        g.precond(F, 2, 0.25, out=out, variant=variant)
    for i in range(3):
        with torch.cuda.stream(s):
            F.copy_(dev(p.F) * (1 + i))
            graph.replay()
            want = ref.precond(F, 2, 0.25, variant=variant)
        s.synchronize()
        assert np.array_equal(host(out), host(want)), i


def test_recovery_is_over_before_the_next_resident_run():
    """A resident run whose tiles need the device for themselves starts only
    when the recovery behind another operator's abort, on another stream, has
    ended too."""
    import torch
    from paper_2006_16861_amd import tdp
    note("resident run behind a recovery")
    p = inputs.random_medium((700, 640), seed=73, width=8)
    # (streams may share a hardware queue, which orders them anyhow: four)
    streams = [torch.cuda.Stream() for _ in range(5)]
    ops, Fs, outs, T = [], [], [], 4
    for s in streams:
        with torch.cuda.stream(s):
            ops.append(tdp.operator_from_problem(p))
            Fs.append(dev(p.F))
            outs.append(ops[-1].precond(Fs[-1], T, 0.25))
    torch.cuda.synchronize()
    want = host(outs[0])
    ops[0].force_resident_abort(True)
    with torch.cuda.stream(streams[0]):
        ops[0].precond(Fs[0], T, 0.25, out=outs[0])
        over = torch.cuda.Event()
        over.record()
    early = []
    for i in range(1, 5):
        with torch.cuda.stream(streams[i]):
            ops[i].precond(Fs[i], T, 0.25, out=outs[i])
        streams[i].synchronize()
        early.append(not over.query())
    torch.cuda.synchronize()
    assert not any(early), early
    assert rel(host(outs[0]), want) <= 1e-13
    for i in range(1, 5):
        assert np.array_equal(host(outs[i]), want) and ops[i].resident_aborts == 0


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
def test_callers_capture_of_a_first_call_27_points(prec, variant):
    """3-D tables with corner entries: the first call of all may be captured
    (use_graph = 0), with one step per launch, which needs no second field pair;
    an eager call after it is the same, bit for bit, with two."""
    import torch
    from paper_2006_16861_amd import tdp
    note(f"capture of a first 27-point call, prec {prec} variant {variant}")
    p = inputs.random_medium((100, 100, 100), seed=83, width=2)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g, ref = (tdp.operator_from_problem(p, scheme="q1", prec=prec) for _ in range(2))
        g.set_tuning(use_graph=0)
        ref.set_tuning(kernel=3, tb_depth=8, tile=0)
        F = dev(p.F)
        out = torch.empty_like(F)
        if variant:
            g.set_tuning(kernel=3, tb_depth=8, tile=0)     # makes the complex fields
            g.precond(F, 1, 0.25, variant=1)
            g.set_tuning(use_graph=0)
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        g.precond(F, 1, 0.25, out=out, variant=variant)
    for i in range(3):
        with torch.cuda.stream(s):
            F.copy_(dev(p.F) * (1 + i))
            graph.replay()
            want = ref.precond(F, 1, 0.25, variant=variant)
            eager = g.precond(F, 1, 0.25, variant=variant)
        s.synchronize()
        assert torch.equal(out, want) and torch.equal(eager, want), i


def test_small_operators_overlap_on_their_streams():
    """Two operators of 200 x 200 nodes (48 tiles each) on two streams: their
    resident runs fit the device together and overlap, instead of taking the
    time of one after the other."""
    import torch
    from paper_2006_16861_amd import tdp
    note("two small operators on two streams")
    p = inputs.random_medium((200, 200), seed=72, width=6)
    # (streams may share a hardware queue, which orders them anyhow: four pairs)
    streams = [torch.cuda.Stream() for _ in range(5)]
    ops, Fs, outs = [], [], []
    for s in streams:
        with torch.cuda.stream(s):
            ops.append(tdp.operator_from_problem(p))
            Fs.append(dev(p.F))
            outs.append(torch.empty_like(Fs[-1]))
    T = 2000 // ops[0].nP

    def ms(*which):
        torch.cuda.synchronize()
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        first, last = streams[which[0]], streams[which[-1]]
        e[0].record(first)
        last.wait_event(e[0])
        for _ in range(8):
            for i in which:
                with torch.cuda.stream(streams[i]):
                    ops[i].precond(Fs[i], T, 0.25, out=outs[i])
        first.wait_stream(last)
        e[1].record(first)
        torch.cuda.synchronize()
        return e[0].elapsed_time(e[1])

    for i in range(5):
        ms(i)
    one = min(ms(0) for _ in range(5))
    both = [min(ms(0, i) for _ in range(3)) for i in range(1, 5)]
    note(f"  one {one:.2f} ms, two {', '.join('%.2f' % b for b in both)} ms")
    assert all(torch.equal(outs[0], U) for U in outs)
    assert all(g.resident_aborts == 0 for g in ops)
    assert min(both) <= 1.5 * one, (one, both)


def test_operators_of_all_sizes_on_their_streams():
    """Runs of one tile per compute unit or less beside each other and beside
    ones that need the device for themselves, from five streams in turn: each
    is bit for bit what the operator gives alone, and none gives up."""
    import torch
    from paper_2006_16861_amd import tdp
    note("operators of all sizes on five streams")
    sizes = [(200, 200), (1000, 1050), (300, 260), (512, 512), (65, 64)]
    ops, Fs, want = [], [], []
    streams = [torch.cuda.Stream() for _ in sizes]
    for i, (n, s) in enumerate(zip(sizes, streams)):
        p = inputs.random_medium(n, seed=78 + i, width=6)
        with torch.cuda.stream(s):
            ops.append(tdp.operator_from_problem(p, prec=i % 2))
            Fs.append(dev(p.F))
            want.append(ops[-1].precond(Fs[-1], 6, 0.25))
        s.synchronize()
    got = []
    for _ in range(12):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                got.append((i, ops[i].precond(Fs[i], 6, 0.25)))
    torch.cuda.synchronize()
    for i, U in got:
        assert torch.equal(U, want[i]), sizes[i]
    assert all(g.resident_aborts == 0 for g in ops)


def test_stream_with_a_part_of_the_compute_units():
    """A stream created with a mask of compute units holds fewer tiles than the
    device: the blocked sweep runs on it, bit for bit, not a resident one that
    gives up and is redone.  A mask of all compute units changes nothing."""
    import ctypes

    import torch
    from paper_2006_16861_amd import tdp
    note("stream with a mask of compute units")
    p = inputs.random_medium((700, 640), seed=84, width=8)
    F = dev(p.F)
    ref = tdp.operator_from_problem(p)
    resident = ref.precond(F, 4, 0.25)
    ref.set_tuning(kernel=2, tb_depth=8, tile=5)
    blocked = ref.precond(F, 4, 0.25)
    torch.cuda.synchronize()
    assert not torch.equal(resident, blocked)       # rounding tells them apart
    hip = ctypes.CDLL("libamdhip64.so")
    words = 8
    for cus, want in ((64, blocked), (256, resident)):
        mask = (ctypes.c_uint32 * words)(*[0xFFFFFFFF if 32 * i < cus else 0 for i in range(words)])
        h = ctypes.c_void_p()
        assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(h), words, mask) == 0
        s = torch.cuda.ExternalStream(h.value)
        with torch.cuda.stream(s):
            g = tdp.operator_from_problem(p)
            got = [g.precond(F, 4, 0.25) for _ in range(2)]
            s.synchronize()
            aborts = g.resident_aborts
            g.close()
        note(f"  {cus} compute units: distance {rel(host(got[0]), host(want)):.1e}, aborts {aborts}")
        assert all(torch.equal(U, want) for U in got) and aborts == 0
        assert hip.hipStreamDestroy(h) == 0
