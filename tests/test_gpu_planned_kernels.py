"""Which kernel the untuned choice takes, at sizes where tests of one of them
depend on it."""
import pytest

pytestmark = pytest.mark.gpu


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
        assert planned((64, 64, 95), prec, scheme="q1") == 1
        assert planned((64, 64, 95), prec, 1, scheme="q1") == 4
        assert planned((64, 64, 97), prec, scheme="q1") == 4
        assert planned((148, 146, 147), prec, scheme="q1") == (4 if prec else 3)
        assert planned((9, 8, 7), prec, 1, damping="cell") == 1
