"""The resident sweep as the library's own choice (2-D, node damping, no tuning
set): grids of exactly one tile and one node more on either axis, both parts
of Definition 4 side by side, a run handed over between launches, the
recovery behind an asynchronous application, and several threads whose
launches must not overlap.  FP64 against the oracle at 1e-10 (the bar of every
FP64 parity test); FP32 against the blocked sweep, whose operations it repeats
in the same order: equal."""
import sys
import threading

import numpy as np
import pytest

import oracle
from paper_2006_16861_amd import inputs

pytestmark = pytest.mark.gpu

TOL64 = 1e-10


def dev(a):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


def host(t):
    return t.detach().cpu().numpy()


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / max(np.linalg.norm(b.ravel()), 1e-300))


# one tile (48 or 64 rows, 64 columns) and its neighbours; many small tiles
SHAPES = [(1, 1), (48, 64), (49, 64), (64, 64), (65, 64), (64, 65), (48, 65), (129, 130), (257, 190)]


@pytest.mark.parametrize("n", SHAPES)
def test_default_sweep_matches_oracle(n):
    from paper_2006_16861_amd import tdp
    p = inputs.random_medium(n, seed=61, width=min(4, min(n) // 4))
    g, o = tdp.operator_from_problem(p), oracle.Op.from_problem(p)
    print(f"[case] default sweep {n}", file=sys.stderr, flush=True)
    assert rel(host(g.precond(dev(p.F), 3, 0.25)), o.precond(p.F, 3, 0.25)) <= TOL64
    assert rel(host(g.precond(dev(p.F), 3, 0.25, variant=1)),
               o.precond(p.F, 3, 0.25, variant=1)) <= TOL64
    g32 = tdp.operator_from_problem(p, prec=tdp.F32)
    for variant in (0, 1):
        U = host(g32.precond(dev(p.F), 3, 0.25, variant=variant))
        g32.set_tuning(kernel=2, tb_depth=4, tile=5)
        assert np.array_equal(U, host(g32.precond(dev(p.F), 3, 0.25, variant=variant)))
        g32.set_tuning()


@pytest.mark.parametrize("n", [(33, 130), (430, 430), (450, 470), (512, 512), (560, 600), (700, 640)])
def test_tile_shapes(n):
    """Every exchange depth where the tile shape changes with the grid: 32-row
    tiles (430 x 430: the last that fit at depth 8), one 48- or 64-row tile per
    compute unit, two.  FP64 against the blocked sweep at 1e-13, the bar of the
    other kernel against kernel comparisons; FP32 equal to it."""
    from paper_2006_16861_amd import tdp
    p = inputs.random_medium(n, seed=67, width=4)
    print(f"[case] tile shapes {n}", file=sys.stderr, flush=True)
    for prec in (tdp.F64, tdp.F32):
        g = tdp.operator_from_problem(p, prec=prec)
        for variant in (0, 1):
            g.set_tuning(kernel=2, tb_depth=4, tile=5)
            U = host(g.precond(dev(p.F), 2, 0.25, variant=variant))
            for k in (2, 4, 6, 8):
                g.set_tuning(kernel=5, tb_depth=k)
                V = host(g.precond(dev(p.F), 2, 0.25, variant=variant))
                if prec == tdp.F32:
                    assert np.array_equal(U, V), (variant, k)
                else:
                    assert rel(V, U) <= 1e-13, (variant, k)
        assert g.resident_aborts == 0


@pytest.mark.parametrize("n,variant", [((60, 50), 0), ((60, 130), 0), ((60, 130), 1)])
def test_runs_longer_than_one_launch(n, variant):
    """N_s = 4104 steps: two launches (4096 + 8)."""
    from paper_2006_16861_amd import tdp
    p = inputs.random_medium(n, seed=62, width=5)
    g, o = tdp.operator_from_problem(p), oracle.Op.from_problem(p)
    T = -(-4097 // g.nP)
    U = host(g.precond(dev(p.F), T, 0.1, variant=variant))
    assert rel(U, o.precond(p.F, T, 0.1, variant=variant)) <= TOL64


@pytest.mark.parametrize("variant", [0, 1])
def test_recovery_behind_an_asynchronous_application(variant):
    """Every wait gives up after a few polls (forced from the host; all kernels
    exit normally): the application is redone behind the run on the stream, and
    the next calls take the blocked sweep."""
    from paper_2006_16861_amd import tdp
    p = inputs.random_medium((150, 140), seed=63, width=4)
    g, o = tdp.operator_from_problem(p), oracle.Op.from_problem(p)
    Uo = o.precond(p.F, 2, 0.25, variant=variant)
    g.force_resident_abort(True)
    assert rel(host(g.precond(dev(p.F), 2, 0.25, variant=variant)), Uo) <= TOL64
    assert rel(host(g.precond(dev(p.F), 2, 0.25, variant=variant)), Uo) <= TOL64
    assert g.resident_aborts == 1
    Ug, ig = g.solve(dev(p.F), T=p.periods, restart=6, fixed_iters=3)
    Uog, _ = o.gmres(p.F, T=p.periods, restart=6, fixed_iters=3)
    assert rel(host(Ug), Uog) <= TOL64 and g.resident_aborts == 1


def test_threads_on_their_own_streams():
    """Launches that together exceed the device's workgroups, from three
    threads: ordered one behind the other, none gives up."""
    import torch
    from paper_2006_16861_amd import tdp
    out = {}

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            p = inputs.random_medium((700 + 20 * i, 640), seed=64 + i, width=8)
            g = tdp.operator_from_problem(p)
            F = dev(p.F)
            got = [g.precond(F, 3, 0.25) for _ in range(6)]
            g.set_tuning(kernel=2, tb_depth=8, tile=5)
            ref = g.precond(F, 3, 0.25)
            torch.cuda.current_stream().synchronize()
            out[i] = (max(rel(host(U), host(ref)) for U in got), g.resident_aborts)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert len(out) == 3 and all(e <= 1e-13 and a == 0 for e, a in out.values()), out
