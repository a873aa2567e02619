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
