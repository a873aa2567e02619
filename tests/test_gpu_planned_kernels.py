"""Which kernel the untuned choice takes, at sizes where tests of one of them
depend on it, and those tests where they did not reach it: the streamed 2-D
sweep's strip edges in FP32, and the resident sweep handed over between launches
in FP32 and under an explicit kernel 5."""
import sys

import numpy as np
import pytest

import oracle
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


def planned(n, prec, variant=0, **kw):
    import torch
    from paper_2006_16861_amd import tdp
    c = torch.ones(n, dtype=torch.float64, device="cuda")
    return tdp.Operator(c, None, 2.0, 0.1, prec=prec, **kw).planned_kernel(variant)


def test_rules():
    for prec in (0, 1):
        # resident where it fits (in FP32 beyond 13 * 2^17 nodes), then, in
        # FP64, blocked, then streamed
        for n in ((1, 1), (64, 64), (65, 64), (512, 512), (1024, 1024)):
            assert planned(n, prec) == 5 and planned(n, prec, 1) == 5, (n, prec)
        assert planned((1300, 1300), prec) == (5 if prec else 2)
        assert planned((1450, 1400), prec) == 6 and planned((2999, 2503), prec, 1) == 6
        # few rows leave the streamed sweep few runs, and FP32 tiles many rows
        assert planned((11, 155000), prec) == (6 if prec else 2)
        assert planned((30, 60000), prec) == (6 if prec else 2)
        assert planned((1340, 1340), prec) == 2 and planned((100, 18000), prec) == (2 if prec else 6)
        assert planned((1500, 1500), prec) == 6 and planned((1600, 1600), prec) == (2 if prec else 6)
        assert planned((1024, 1024), prec, scheme="q1") == 2
        assert planned((1024, 1024), prec, 1, damping="cell") == 2
        # 3-D: two steps per launch; corner entries by size and form
        assert planned((64, 64, 64), prec) == 4 and planned((9, 8, 7), prec, scheme="fd2") == 4
        for n in ((1, 4, 6), (1, 300, 300), (2, 7, 2), (3, 64, 64)):      # few planes
            assert planned(n, prec) == (4 if prec else 1), n
            assert planned(n, prec, 1) == (4 if prec else 1), n
        assert planned((2, 200, 200), prec) == 4 and planned((4, 4, 4), prec) == 4
        assert planned((62, 64, 64), prec, scheme="q1") == 1
        assert planned((62, 64, 64), prec, 1, scheme="q1") == 4
        assert planned((64, 64, 97), prec, scheme="q1") == (1 if prec else 4)
        assert planned((148, 146, 147), prec, scheme="q1") == (4 if prec else 3)
        for variant in (0, 1):
            # narrow rows; where two steps per launch take longer than one; where not
            assert planned((110, 216, 3), prec, variant, scheme="q1") == 4
            assert planned((133, 106, 85), prec, variant, scheme="q1") == (4 if prec else 3)
            assert planned((165, 125, 135), prec, variant, scheme="q1") == 3
            assert planned((111, 107, 93), prec, variant, scheme="q1") == 4
            assert planned((131, 150, 117), prec, variant, scheme="q1") == 4
            assert planned((137, 182, 101), prec, variant, scheme="q1") == 4
        assert planned((9, 8, 7), prec, 1, damping="cell") == 1


@pytest.mark.parametrize("n", [(1, 4, 6), (1, 60, 70), (2, 7, 2), (3, 20, 20), (1, 1, 1), (4, 5, 6)])
def test_few_planes_match_the_oracle(n):
    """The untuned kernel on 3-D grids of few planes, both forms, at the FP64 bar."""
    from paper_2006_16861_amd import tdp
    print(f"[case] few planes {n}", file=sys.stderr, flush=True)
    p = inputs.random_medium(n, seed=87, width=min(1, min(n) // 2))
    g, o = tdp.operator_from_problem(p), oracle.Op.from_problem(p)
    for variant in (0, 1):
        U = host(g.precond(dev(p.F), 3, 0.25, variant=variant))
        assert rel(U, o.precond(p.F, 3, 0.25, variant=variant)) <= 1e-10, variant


@pytest.mark.parametrize("n", [(9000, 20), (297, 657), (16 * 256, 48), (16 * 256 + 1, 48)])
def test_cell_damping_tile_on_long_grids(n):
    """FP32 with the cell damping: the untuned tile is the one of few rows only
    where its tiles are at most the compute units (256 and 257 of them).  The
    same results as on 64 x 64 tiles, bit for bit, in no more time."""
    import torch
    from paper_2006_16861_amd import tdp
    p = inputs.random_medium(n, seed=88, width=4)
    g = tdp.operator_from_problem(p, prec=1, damping="cell")
    F = dev(p.F)
    out = torch.empty_like(F)

    def ms():
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(4):
            g.precond(F, 10, 0.25, out=out, variant=1)
        e[1].record()
        torch.cuda.synchronize()
        return e[0].elapsed_time(e[1])

    t = {}
    for name, tun in (("tile 4", dict(kernel=2, tb_depth=8, tile=4)), ("untuned", {})):
        g.set_tuning(**tun)
        ms()
        t[name] = min(ms() for _ in range(5))
        t[name + " U"] = host(out)
    print(f"[case]   cell damping {n}: {t['tile 4']:.3f} ms, untuned {t['untuned']:.3f}", file=sys.stderr, flush=True)
    assert np.array_equal(t["tile 4 U"], t["untuned U"])
    assert t["untuned"] <= 1.2 * t["tile 4"]


# the shapes of the streamed sweep's edges, as each precision reaches them
# (FP32's tiles of 64 x 64 hold more than FP64's of 48 x 64)
EDGES = [((27100, 63), 0), ((26700, 64), 0), ((15400, 111), 0), ((15301, 112), 0),
         ((40000, 63), 1), ((40000, 64), 1), ((20500, 111), 1), ((20500, 112), 1),
         ((2, 860000), 0), ((2, 860000), 1), ((10, 175000), 0), ((19, 92500), 0),
         ((11, 155000), 1), ((1450, 1400), 0), ((1450, 1400), 1)]


@pytest.mark.parametrize("n,prec", EDGES)
def test_streamed_sweep_runs_at_its_edges(n, prec):
    """FP64 against the blocked sweep at 1e-13, FP32 equal to it; N_s = 9 to 27."""
    from paper_2006_16861_amd import tdp
    print(f"[case] streamed sweep {n} prec {prec}", file=sys.stderr, flush=True)
    p = inputs.random_medium(n, seed=85, width=min(2, min(n) // 2))
    g = tdp.operator_from_problem(p, prec=prec)
    assert g.planned_kernel(0) == 6 and g.planned_kernel(1) == 6
    F = dev(p.F)
    for T, variant in ((1, 0), (3, 0), (2, 1)):
        g.set_tuning(kernel=2, tb_depth=4, tile=5)
        U = host(g.precond(F, T, 0.25, variant=variant))
        g.set_tuning()
        V = host(g.precond(F, T, 0.25, variant=variant))
        if prec:
            assert np.array_equal(U, V), (T, variant)
        else:
            assert rel(V, U) <= 1e-13, (T, variant)


@pytest.mark.parametrize("kernel", [0, 5])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nP", [12, 13])
def test_resident_runs_handed_over(nP, prec, kernel):
    """More than 4096 steps: two launches, the second of an odd number of steps
    (n_P = 13: 4121 = 4096 + 25), several tiles.  Against the blocked sweep:
    FP64 at 1e-11 (it drifts from it by rounding over 4000 steps; the oracle's
    bar is 1e-10), FP32 equal; FP64 also against the oracle."""
    from paper_2006_16861_amd import tdp
    p = inputs.random_medium((60, 130), seed=86, width=5)
    T = {12: 342, 13: 317}[nP]
    print(f"[case] {T * nP} steps, prec {prec}, kernel {kernel}", file=sys.stderr, flush=True)
    g = tdp.Operator(dev(p.c), dev(p.R), p.omega, p.h, prec=prec, steps_per_period=nP)
    F = dev(p.F)
    for variant in (0, 1):
        g.set_tuning(kernel=2, tb_depth=8, tile=8 if prec else 5)
        U = host(g.precond(F, T, 0.1, variant=variant))
        g.set_tuning(kernel=kernel, tb_depth=4 if kernel else 0)
        assert g.planned_kernel(variant) == 5
        V = host(g.precond(F, T, 0.1, variant=variant))
        if prec:
            assert np.array_equal(U, V), variant
        else:
            assert rel(V, U) <= 1e-11, variant
            o = oracle.Op.from_problem(p, nP=nP)
            assert rel(V, o.precond(p.F, T, 0.1, variant=variant)) <= 1e-10
    assert g.resident_aborts == 0
