"""Which resident launches may overlap (csrc/res_gate.h, host code only): over
random sequences of launches and destroyed operators, no set of launches that
may run at the same time needs more than the device has, unless it is a single
launch; small launches of several operators are not ordered at all."""
import ctypes
import itertools
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include "res_gate.h"
using tdp::ResGateBook;
extern "C" {
ResGateBook *book_new() { return new ResGateBook; }
void book_free(ResGateBook *b) { delete b; }
int book_admit(ResGateBook *b, unsigned long long op, int need, int cap, unsigned long long *wait)
{
    void *w[ResGateBook::kMax];
    const int n = b->admit(op, (void *)op, need, cap, w);
    for (int i = 0; i < n; ++i) wait[i] = (unsigned long long)w[i];
    return n;
}
void book_forget(ResGateBook *b, unsigned long long op) { b->forget(op); }
int book_units(int n) { return ResGateBook::units(n); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("gate")
    (d / "gate.cpp").write_text(SRC)
    so = str(d / "gate.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2006_16861_amd", "csrc"),
                           str(d / "gate.cpp"), "-o", so])
    L = ctypes.CDLL(so)
    L.book_new.restype = ctypes.c_void_p
    L.book_free.argtypes = [ctypes.c_void_p]
    L.book_admit.argtypes = [ctypes.c_void_p, ctypes.c_ulonglong, ctypes.c_int, ctypes.c_int,
                             ctypes.POINTER(ctypes.c_ulonglong)]
    L.book_forget.argtypes = [ctypes.c_void_p, ctypes.c_ulonglong]
    return L


class Model:
    """Launches with the launches that each is ordered behind."""

    def __init__(self, lib, cap):
        self.lib, self.cap, self.b = lib, cap, lib.book_new()
        self.last, self.behind, self.need, self.done = {}, [], [], set()

    def launch(self, op, need):
        buf = (ctypes.c_ulonglong * 64)()
        n = self.lib.book_admit(self.b, op, need, self.cap, buf)
        before = set()
        for o in list(buf[:n]) + [op]:
            if o in self.last:
                before |= self.behind[self.last[o]] | {self.last[o]}
        self.last[op] = len(self.need)
        self.behind.append(before)
        self.need.append(need)
        return n

    def destroy(self, op):
        """The operator's stream is waited for first."""
        if op in self.last:
            self.done |= self.behind[self.last[op]] | {self.last.pop(op)}
        self.lib.book_forget(self.b, op)

    def overlapping(self):
        live = [i for i in range(len(self.need)) if i not in self.done]
        for k in range(2, len(live) + 1):
            any_ = False
            for c in itertools.combinations(live, k):
                if all(i not in self.behind[j] and j not in self.behind[i]
                       for i, j in itertools.combinations(c, 2)):
                    any_ = True
                    yield c
            if not any_:
                return


@pytest.mark.parametrize("seed", range(60))
def test_overlapping_launches_fit_the_device(lib, seed):
    rng = random.Random(seed)
    m = Model(lib, 8)
    for _ in range(11):
        op = rng.randint(1, 5)
        if rng.random() < 0.15:
            m.destroy(op)
        else:
            m.launch(op, rng.choice([1, 1, 2, 3, 5, 8, 16]))
    for c in m.overlapping():
        assert sum(m.need[i] for i in c) <= 8, (c, m.need, m.behind)
    lib.book_free(m.b)


def test_small_launches_are_not_ordered(lib):
    m = Model(lib, 8)
    for _ in range(4):
        for op in (1, 2, 3):
            assert m.launch(op, 2) == 0
    assert m.launch(4, 3) == 3 and m.launch(4, 3) == 0 and m.launch(1, 2) == 2
    lib.book_free(m.b)


def test_units(lib):
    assert [lib.book_units(n) for n in (1, 32, 33, 48, 256, 257, 494)] == [1, 1, 2, 2, 8, 9, 16]
