"""The streamed 2-D sweep (the untuned default of large grids that do not fit the
resident tiles) at its edges: 63 columns are one strip, 64 two, 111 / 112 the
last of two and the first of three; runs of two rows, of ten, and a last run
shorter than the others; few rows and many strips; samples inside a launch and
steps left over for the blocked tile (N_s = 9 to 27).  FP64 against the blocked
sweep at 1e-13, the bar of the other kernel against kernel comparisons; FP32,
whose operations are the same in the same order, equal to it."""
import sys

import numpy as np
import pytest

from paper_2006_16861_amd import inputs

pytestmark = pytest.mark.gpu

# at least 13 * 2^17 nodes each, more than the resident tiles hold
SHAPES = [(27100, 63), (26700, 64), (15400, 111), (15301, 112), (2, 860000), (11, 155000), (1450, 1400)]


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
def test_streamed_sweep_at_its_edges(n):
    from paper_2006_16861_amd import tdp
    print(f"[case] streamed sweep {n}", file=sys.stderr, flush=True)
    p = inputs.random_medium(n, seed=81, width=min(2, min(n) // 2))
    for prec in (tdp.F64, tdp.F32):
        g = tdp.operator_from_problem(p, prec=prec)
        F = dev(p.F)
        for T, variant in ((1, 0), (3, 0), (2, 1)):
            g.set_tuning(kernel=2, tb_depth=4, tile=5)
            U = host(g.precond(F, T, 0.25, variant=variant))
            g.set_tuning()
            V = host(g.precond(F, T, 0.25, variant=variant))
            if prec == tdp.F32:
                assert np.array_equal(U, V), (T, variant)
            else:
                assert rel(V, U) <= 1e-13, (T, variant)
