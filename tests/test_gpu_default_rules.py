"""The untuned kernel of the 3-D tables with corner entries and of the 2-D cell
damping on either side of each size at which it changes: the same results, bit
for bit, as the kernel that every size took (one step per launch on 8 x 64 columns;
the 32 x 64 or, in FP32, the 64 x 64 I_abd tile at depth 8)."""
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


# below and above 3 * 2^17 and 3 * 2^20 nodes, and the smallest
@pytest.mark.parametrize("n", [(3, 2, 5), (64, 64, 95), (64, 64, 97), (146, 146, 147), (148, 146, 147)])
def test_corner_tables_3d(n):
    from paper_2006_16861_amd import tdp
    print(f"[case] untuned 27-point sweep {n}", file=sys.stderr, flush=True)
    p = inputs.random_medium(n, seed=91, width=min(2, min(n) // 2))
    for prec in (tdp.F64, tdp.F32):
        g = tdp.operator_from_problem(p, prec=prec, scheme="q1")
        for T, variant in ((2, 0), (1, 1)):
            g.set_tuning(kernel=3, tb_depth=8, tile=0)
            U = host(g.precond(dev(p.F), T, 0.25, variant=variant))
            g.set_tuning()
            assert np.array_equal(host(g.precond(dev(p.F), T, 0.25, variant=variant)), U), variant


# below and above 3 * 2^16 and 3 * 2^19 nodes, and the smallest
@pytest.mark.parametrize("n", [(5, 4), (440, 446), (444, 444), (1254, 1254), (1255, 1254)])
def test_cell_damping_2d(n):
    from paper_2006_16861_amd import tdp
    print(f"[case] untuned cell damping {n}", file=sys.stderr, flush=True)
    p = inputs.random_medium(n, seed=92, width=min(4, min(n) // 2))
    for prec in (tdp.F64, tdp.F32):
        g = tdp.operator_from_problem(p, prec=prec, damping="cell")
        g.set_tuning(kernel=2, tb_depth=8, tile=7 if prec == tdp.F64 else 4)
        U = host(g.precond(dev(p.F), 2, 0.25, variant=1))
        g.set_tuning()
        assert np.array_equal(host(g.precond(dev(p.F), 2, 0.25, variant=1)), U)
