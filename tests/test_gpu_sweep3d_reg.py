"""The two-step 3-D sweep with the rows in registers (kernel 4 and the untuned
default for tables without corner entries) at the edges of its tiles: 64 columns
are one tile and 65 two, 112 / 113, 120 / 121 and 124 / 125 columns change the
column step or the count; 16 rows are one tile (32 in FP32 tile 2), each 14 (30)
more another; runs of two planes, of one, and a grid of one plane.  FP64 against
the oracle at 1e-10 (the bar of every FP64 parity test).  FP32 differs from
FP64 fields by at most 1e-4 (the bar of the FP32 parity tests), and its two tile
shapes, which do the same operations on each node, must be equal."""
import sys

import numpy as np
import pytest

import oracle
from paper_2006_16861_amd import inputs

pytestmark = pytest.mark.gpu

# every column and row edge with few planes; odd ones
SHAPES = [(1, 1, 1), (2, 16, 63), (3, 17, 64), (4, 15, 65), (5, 30, 112), (3, 31, 113), (2, 32, 120),
          (6, 33, 121), (3, 45, 124), (4, 62, 125), (33, 14, 61), (2, 63, 185)]


def dev(a):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


def host(t):
    return t.detach().cpu().numpy()


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / max(np.linalg.norm(b.ravel()), 1e-300))


@pytest.mark.parametrize("n", SHAPES)
def test_register_sweep_at_tile_edges(n):
    from paper_2006_16861_amd import tdp
    print(f"[case] register sweep {n}", file=sys.stderr, flush=True)
    p = inputs.random_medium(n, seed=71, width=min(2, min(n) // 2))
    g, o = tdp.operator_from_problem(p), oracle.Op.from_problem(p)
    g32 = tdp.operator_from_problem(p, prec=tdp.F32)
    for T, variant in ((3, 0), (2, 1)):
        U = o.precond(p.F, T, 0.25, variant=variant)
        for tuning in ({}, {"kernel": 4, "tb_depth": 1}, {"kernel": 4, "tb_depth": 64}):
            g.set_tuning(**tuning)
            assert rel(host(g.precond(dev(p.F), T, 0.25, variant=variant)), U) <= 1e-10, tuning
        g32.set_tuning()
        V = host(g32.precond(dev(p.F), T, 0.25, variant=variant))
        assert rel(V, U) <= 1e-4
        for tile in (0, 2):
            g32.set_tuning(kernel=4, tb_depth=3, tile=tile)
            assert np.array_equal(host(g32.precond(dev(p.F), T, 0.25, variant=variant)), V), tile
