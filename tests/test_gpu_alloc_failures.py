"""Allocations that fail (simulated: a preloaded function refuses requests of a
given size a given number of times).  The call returns TDP_ENOMEM with nothing
written, and a later one, with memory there again, is right: nothing half made
is taken for whole."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
static size_t g_size;
static int g_skip, g_times, g_host;
void shim_fail(int host, size_t size, int skip, int times)
{
    g_host = host; g_size = size; g_skip = skip; g_times = times;
}
int shim_left(void) { return g_times; }
static int refuse(int host, size_t size)
{
    if (host != g_host || size != g_size || g_times == 0) return 0;
    if (g_skip > 0) { --g_skip; return 0; }
    --g_times;
    return 1;
}
static void *real(const char *name)          /* the runtime is loaded, but not globally */
{
    void *h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    if (!h) h = dlopen("libamdhip64.so", RTLD_LAZY | RTLD_NOLOAD);
    return h ? dlsym(h, name) : NULL;
}
int hipMalloc(void **p, size_t size)
{
    int (*f)(void **, size_t) = (int (*)(void **, size_t))real("hipMalloc");
    return !f || refuse(0, size) ? 2 : f(p, size);
}
int hipHostMalloc(void **p, size_t size, unsigned flags)
{
    int (*f)(void **, size_t, unsigned) = (int (*)(void **, size_t, unsigned))real("hipHostMalloc");
    return !f || refuse(1, size) ? 2 : f(p, size, flags);
}
"""

CHILD = r"""
import ctypes, sys
import torch
from paper_2006_16861_amd import inputs, tdp
shim = ctypes.CDLL(sys.argv[1])
shim.shim_fail.argtypes = [ctypes.c_int, ctypes.c_size_t, ctypes.c_int, ctypes.c_int]

def rel(a, b):
    return float((a - b).norm() / b.norm())

def refused(name, host, size, skip, make, call, ref):
    print("[case]", name, flush=True)
    g = make()
    shim.shim_fail(host, size, skip, 1)
    try:
        call(g)
    except tdp.TdpError as e:
        assert e.code == tdp.ENOMEM, (name, str(e))
    else:
        raise AssertionError(name + ": not refused")
    assert shim.shim_left() == 0, name
    torch.cuda.synchronize()
    for _ in range(2):
        out = call(g)
        torch.cuda.synchronize()
        assert rel(out, ref) <= 1e-11, (name, rel(out, ref))

p = inputs.random_medium((150, 140), seed=81, width=4)
F = torch.as_tensor(p.F, device="cuda")
N = F.numel()
op = lambda **kw: tdp.operator_from_problem(p, **kw)
ref = op()
ref.set_tuning(kernel=2, tb_depth=4, tile=5)
U0, U1 = ref.precond(F, 2, 0.25), ref.precond(F, 2, 0.25, variant=1)
S = ref.solve(F, T=2, restart=5, fixed_iters=4)[0]

def tuned(kernel):
    def make():
        g = op()
        g.set_tuning(kernel=kernel)
        return g
    return make

pre = lambda g: g.precond(F, 2, 0.25)
pre1 = lambda g: g.precond(F, 2, 0.25, variant=1)
sol = lambda g: g.solve(F, T=2, restart=5, fixed_iters=4)[0]
refused("pinned word of the resident sweep", 1, 8, 0, op, pre, U0)
for skip in (0, 1):
    refused(f"field pair {skip}, blocked", 0, 8 * N, skip, tuned(2), pre, U0)
    refused(f"field pair {skip}, resident", 0, 8 * N, skip, op, pre, U0)
    refused(f"complex fields {skip}", 0, 16 * N, skip, op, pre1, U1)
refused("krylov basis", 0, 16 * N * 6, 0, op, sol, S)
for skip in range(4):
    refused(f"work vector {skip}", 0, 16 * N, skip, op, sol, S)
refused("krylov coefficients", 0, 8 * 8 * 7, 0, op, sol, S)
refused("krylov coefficients, pinned", 1, 8 * 8 * 7, 0, op, sol, S)

# 27-point tables in 3-D: one step per launch without the second field pair
# (the same results, bit for bit), two with it
p = inputs.random_medium((100, 100, 100), seed=82, width=2)
F = torch.as_tensor(p.F, device="cuda")
for prec in (0, 1):
    g = tdp.operator_from_problem(p, scheme="q1", prec=prec)
    g.set_tuning(kernel=3, tb_depth=8, tile=0)
    want = [g.precond(F, 2, 0.25, variant=v) for v in (0, 1)]
    for skip in (0, 1):
        print("[case] field pair", skip, "of the 27-point sweep, prec", prec, flush=True)
        g = tdp.operator_from_problem(p, scheme="q1", prec=prec)
        for v in (0, 1):
            shim.shim_fail(0, (4 if prec else 8) * F.numel(), skip, 1)
            assert torch.equal(g.precond(F, 2, 0.25, variant=v), want[v])
            assert shim.shim_left() == 0
        for v in (0, 1):
            assert torch.equal(g.precond(F, 2, 0.25, variant=v), want[v])
print("done", flush=True)
"""


def test_failed_allocations_leave_nothing_half_made(tmp_path):
    (tmp_path / "shim.c").write_text(SHIM)
    so = str(tmp_path / "shim.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", str(tmp_path / "shim.c"), "-o", so, "-ldl"])
    env = dict(os.environ)
    env["LD_PRELOAD"] = (env["LD_PRELOAD"] + ":" if env.get("LD_PRELOAD") else "") + so
    r = subprocess.run([sys.executable, "-u", "-c", CHILD, so], cwd=ROOT, env=env, text=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, timeout=100)
    print(r.stdout, file=sys.stderr, flush=True)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("done"), r.stdout[-1500:]
