"""What an abort of the resident sweep costs and how it is accounted for (the abort
is forced from the host; all kernels exit normally), and what an operator keeps
for its runs."""
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


def test_abort_is_counted_once_its_application_is_over():
    import torch
    from paper_2006_16861_amd import tdp
    note("abort counted by the query")
    p = inputs.random_medium((150, 140), seed=74, width=4)
    g = tdp.operator_from_problem(p)
    g.force_resident_abort(True)
    g.precond(dev(p.F), 2, 0.25)
    torch.cuda.synchronize()
    assert g.resident_aborts == 1
    assert g.resident_aborts == 1


def test_set_tuning_brings_the_resident_sweep_back():
    """set_tuning after an abort: the next application runs the resident sweep
    again (and, still forced, aborts again)."""
    import torch
    from paper_2006_16861_amd import tdp
    note("set_tuning after an abort")
    p = inputs.random_medium((150, 140), seed=75, width=4)
    g = tdp.operator_from_problem(p)
    F = dev(p.F)
    g.force_resident_abort(True)
    for i in range(2):
        g.precond(F, 2, 0.25)
        torch.cuda.synchronize()
        g.set_tuning()
    g.precond(F, 2, 0.25)
    torch.cuda.synchronize()
    g.precond(F, 2, 0.25)
    assert g.resident_aborts == 3


def test_every_aborted_application_is_counted():
    """Several asynchronous applications, all aborted before the host looks."""
    import torch
    from paper_2006_16861_amd import tdp
    note("three aborts in flight")
    p = inputs.random_medium((150, 140), seed=75, width=4)
    g = tdp.operator_from_problem(p)
    F = dev(p.F)
    g.precond(F, 2, 0.25)
    torch.cuda.synchronize()
    g.force_resident_abort(True)
    s = torch.cuda.current_stream()
    busy = torch.zeros(1 << 28, device="cuda")
    for _ in range(100):
        busy.add_(1)               # the applications queue up behind this
    for _ in range(3):
        g.precond(F, 2, 0.25)
    s.synchronize()
    assert g.resident_aborts == 3


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,T,variant", [((700, 640), 4, 0), ((700, 640), 4, 1), ((1000, 1050), 3, 0),
                                           ((65, 40), 30, 1), ((33, 130), 31, 0), ((33, 130), 345, 0)])
def test_recovery_is_right_and_takes_a_bounded_multiple_of_the_blocked_sweep(n, T, variant, prec):
    """The recovery is the same recurrence at no more than 20 times the time of
    the blocked sweep: it holds the stream for milliseconds, not seconds."""
    import torch
    from paper_2006_16861_amd import tdp
    note(f"recovery {n} T={T} variant {variant} prec {prec}")
    p = inputs.random_medium(n, seed=76, width=6)
    g = tdp.operator_from_problem(p, prec=prec)
    F = dev(p.F)
    out = torch.empty_like(F)

    def ms():
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        torch.cuda.synchronize()
        e[0].record()
        g.precond(F, T, 0.25, out=out, variant=variant)
        e[1].record()
        torch.cuda.synchronize()
        return e[0].elapsed_time(e[1])

    g.set_tuning(kernel=2, tb_depth=8, tile=8 if prec else 5)
    ms()
    blocked = min(ms() for _ in range(3))
    want = host(out)
    g.set_tuning()
    ms()
    g.force_resident_abort(True)
    redone = ms()
    note(f"  {T * g.nP} steps: blocked {blocked:.3f} ms, aborted and redone {redone:.3f} ms")
    # FP32: the recovery sums the stencil in another order (the bar of the other
    # FP32 kernel against kernel comparisons)
    assert rel(host(out), want) <= (1e-5 if prec else 1e-13)
    assert redone <= 20 * blocked + 1.0, (blocked, redone)


def test_device_tables_stay_bounded():
    """A caller that varies rho: the device copies of the forcing tables are
    bounded, not one more for every value."""
    import torch
    from paper_2006_16861_amd import tdp
    p = inputs.random_medium((60, 50), seed=77, width=4)
    g = tdp.operator_from_problem(p)
    F = dev(p.F)
    out = torch.empty_like(F)
    T = -(-(1 << 16) // g.nP)
    note(f"tables of {T * g.nP} steps")

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    rhos = [0.1 + 0.002 * i for i in range(72)]
    for r in rhos[:24]:
        g.precond(F, T, r, out=out)
    before = free()
    for r in rhos[24:]:
        g.precond(F, T, r, out=out)
    grown = before - free()
    note(f"  {grown / 2**20:.1f} MiB more after {len(rhos) - 24} further tables of 1 MiB")
    assert grown <= 20 << 20
    # an earlier value again, after its table has left
    want = g.precond(F, T, rhos[0]).clone()
    g.set_tuning(kernel=2, tb_depth=4, tile=5)
    assert rel(host(g.precond(F, T, rhos[0])), host(want)) <= 1e-11


def test_new_window_does_not_wait_for_other_streams():
    """An application with a rho that the operator has not seen is as
    asynchronous as one that it has: the host does not wait for work on the
    default stream, nor for the operator's own."""
    import time

    import torch
    from paper_2006_16861_amd import tdp
    note("new rho behind queued work")
    p = inputs.random_medium((150, 140), seed=75, width=4)
    g = tdp.operator_from_problem(p)
    F = dev(p.F)
    out = torch.empty_like(F)
    busy = torch.zeros(1 << 30, device="cuda")

    def seconds(rho):
        torch.cuda.synchronize()
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(60):
            busy.add_(1)
        e[1].record()
        t = time.perf_counter()
        g.precond(F, 2, rho, out=out)
        t = time.perf_counter() - t
        torch.cuda.synchronize()
        return t, 1e-3 * e[0].elapsed_time(e[1])

    seconds(0.25)
    known, queued = seconds(0.25)
    fresh, _ = seconds(0.3)
    note(f"  queued work {queued * 1e3:.1f} ms, host time of a call {known * 1e3:.2f} ms, of one with a new rho {fresh * 1e3:.2f} ms")
    assert queued >= 0.03
    assert fresh <= known + 0.3 * queued


@pytest.mark.parametrize("n", [(60, 50), (150, 140), (700, 640)])
def test_first_call_does_not_wait_for_other_streams(n):
    """Nor does a new operator's first application in either form."""
    import time

    import torch
    from paper_2006_16861_amd import tdp
    note(f"first calls of {n} behind queued work")
    p = inputs.random_medium(n, seed=75, width=4)
    F = dev(p.F)
    out = torch.empty_like(F)
    busy = torch.zeros(1 << 30, device="cuda")
    tdp.operator_from_problem(p).precond(F, 2, 0.25, out=out)
    g = tdp.operator_from_problem(p)
    for variant in (0, 1):
        torch.cuda.synchronize()
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(60):
            busy.add_(1)
        e[1].record()
        t = time.perf_counter()
        g.precond(F, 2, 0.25, out=out, variant=variant)
        t = time.perf_counter() - t
        torch.cuda.synchronize()
        queued = 1e-3 * e[0].elapsed_time(e[1])
        note(f"  variant {variant}: queued work {queued * 1e3:.1f} ms, host time of the call {t * 1e3:.2f} ms")
        assert queued >= 0.03 and t <= 0.3 * queued
