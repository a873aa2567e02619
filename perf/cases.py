"""Performance cases: what a user of the library has it do, through its public entry points.

Each case is one call a program repeats: a preconditioner application (the hot path of every
solve), a GMRES solve, a batched solve, a differentiable solve with its backward pass.  Sizes
follow the repository's own workloads: const2d-64, smooth2d-1024, the uneven batch of
128..768-node axes, smooth2d-512 with several sources, smooth3d-128, layered3d-256, and the
2-D grids beyond the last-level cache.  Operators keep the library's default tuning.

`exact` evaluates the same definitions (Table 1, Definition 4, S_T^abd, GMRES, the gradient of
the squared slowness) with plain torch in 64 bits.
"""
import math

import torch

from paper_2006_16861_amd import autograd, tdp

DEV = "cuda"

# Cell tables (stiffness, mass) of the schemes, entry k for corner pairs that differ in k axes.
TABLES = {
    ("compact", 2): ((5 / 6, -1 / 3, -1 / 6), (1 / 6, 1 / 24, 0.0)),
    ("compact", 3): ((1 / 2, -1 / 12, -1 / 12, 0.0), (1 / 16, 1 / 48, 0.0, 0.0)),
    ("fd2", 2): ((1.0, -0.5, 0.0), (0.25, 0.0, 0.0)),
    ("fd2", 3): ((0.75, -0.25, 0.0, 0.0), (0.125, 0.0, 0.0, 0.0)),
    ("q1", 2): ((2 / 3, -1 / 6, -1 / 3), (1 / 9, 1 / 18, 1 / 36)),
    ("q1", 3): ((1 / 3, 0.0, -1 / 12, -1 / 12), (1 / 27, 1 / 54, 1 / 108, 1 / 216)),
}


def _case(name, kind, n, prec="f64", variant=0, damping="node", scheme="compact", spp=0, ppw=10.0,
          width=32, iters=0, nrhs=1, fields=0):
    n = list(n) + [0] * (3 - len(n))
    return {"name": name, "kind": kind, "n0": n[0], "n1": n[1], "n2": n[2], "prec": prec,
            "variant": variant, "damping": damping, "scheme": scheme, "spp": spp, "ppw": ppw,
            "width": width, "iters": iters, "nrhs": nrhs, "fields": fields}


def listed():
    return [
        # The smallest problem (const2d-64): an interactive call, latency and launches count.
        _case("precond-2d-64", "precond", (64, 64), width=8),
        # An ordinary uneven survey grid with the complex-linear map and the fewest steps per period.
        _case("precond-2d-397x701-def4", "precond", (397, 701), variant=1, spp=-1, ppw=8.0),
        # One application of the headline workload (smooth2d-1024), FP64 and FP32 fields.
        _case("precond-2d-1024", "precond", (1024, 1024)),
        _case("precond-2d-1024-f32", "precond", (1024, 1024), prec="f32"),
        # A grid far beyond what the chip holds, ragged on both axes.
        _case("precond-2d-2999x2503", "precond", (2999, 2503)),
        # Non-diagonal (cell) damping: S_T^abd on the headline grid.
        _case("precond-2d-1024-cell", "precond", (1024, 1024), variant=1, damping="cell"),
        # The 3-D workloads: smooth3d-128 in FP64, layered3d-256 with FP32 fields, and an uneven
        # grid with the full 27-point stencil.
        _case("precond-3d-128", "precond", (128, 128, 128), spp=-1, ppw=8.0, width=16),
        _case("precond-3d-256-f32", "precond", (256, 256, 256), prec="f32", spp=-1, ppw=8.0, width=24),
        _case("precond-3d-131x150x117-q1", "precond", (131, 150, 117), scheme="q1", spp=-1, ppw=8.0,
              width=16),
        # A point-source GMRES solve on the headline grid, stopped after six iterations.
        _case("solve-2d-1024", "solve", (1024, 1024), iters=6),
        # Many sources on one medium and a few uneven problems, FP32 fields, in lockstep.
        _case("batch-512-f32", "batch", (512, 512), prec="f32", iters=2, nrhs=16, fields=8),
        # One gradient of an inversion: forward and adjoint solves of two sources, dL/dm and dL/dF.
        _case("gradient-3d-64", "gradient", (64, 64, 64), spp=-1, ppw=8.0, width=8, nrhs=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["precond2"] * 5 + ["precond3"] * 4 + ["solve", "solve", "batch", "gradient"])
    spp = rng.choice([0, -1])
    ppw = rng.choice([8.0, 10.0])
    prec = rng.choice(["f64", "f32"])
    if kind == "precond2":
        a = _log_int(rng, 48, 2400)
        b = max(48, min(2400, int(a * rng.uniform(0.5, 2.0))))
        damping = rng.choice(["node", "node", "node", "cell"])
        variant = 1 if damping == "cell" else rng.choice([0, 0, 1])
        scheme = rng.choice(["compact", "compact", "compact", "fd2", "q1"])
        return _case("", "precond", (a, b), prec, variant, damping, scheme, spp, ppw,
                     min(32, min(a, b) // 4))
    if kind == "precond3":
        a = _log_int(rng, 32, 256)
        n = [a] + [max(32, min(256, int(a * rng.uniform(0.6, 1.5)))) for _ in range(2)]
        scheme = rng.choice(["compact", "compact", "compact", "fd2", "q1"])
        return _case("", "precond", n, prec, rng.choice([0, 0, 0, 1]), "node", scheme, spp, ppw,
                     max(4, min(24, min(n) // 8)))
    if kind == "solve":
        a = _log_int(rng, 96, 1100)
        b = max(96, min(1100, int(a * rng.uniform(0.6, 1.6))))
        return _case("", "solve", (a, b), "f64", 0, "node", "compact", spp, ppw,
                     min(32, min(a, b) // 4), iters=rng.randint(3, 8))
    if kind == "batch":
        a = _log_int(rng, 128, 600)
        b = max(128, min(600, int(a * rng.uniform(0.6, 1.6))))
        return _case("", "batch", (a, b), prec, 0, "node", "compact", spp, ppw, 32, iters=2,
                     nrhs=rng.randint(4, 20), fields=rng.randint(1, 8))
    n = [rng.randint(36, 72) for _ in range(3)]
    return _case("", "gradient", n, "f64", 0, "node", "compact", -1, ppw, 8,
                 nrhs=rng.randint(1, 3))


# ---------------------------------------------------------------- problems

def _shape(case):
    return tuple(v for v in (case["n0"], case["n1"], case["n2"]) if v)


def _problem(n, seed, ppw, width, cmin=1.5, cmax=4.5):
    """(c, R, omega, h, T): a smooth medium, a quadratic absorbing layer inside the grid, omega
    from `ppw` points per shortest wavelength, T the model's size in wavelengths."""
    g = torch.Generator(device="cpu").manual_seed(seed)
    coarse = torch.randn((1, 1) + tuple(max(3, v // 24) for v in n), generator=g, dtype=torch.float64)
    mode = "bilinear" if len(n) == 2 else "trilinear"
    f = torch.nn.functional.interpolate(coarse.to(DEV), size=n, mode=mode, align_corners=True)
    pool = torch.nn.functional.avg_pool2d if len(n) == 2 else torch.nn.functional.avg_pool3d
    for _ in range(2):      # round the kinks off, so that the extreme speeds are met smoothly
        f = pool(f, 9, stride=1, padding=4, count_include_pad=False)
    f = f[0, 0]
    c = (cmin + (cmax - cmin) * (f - f.min()) / (f.max() - f.min())).contiguous()
    h = 1.0 / (max(n) + 1)
    omega = 2.0 * math.pi * cmin / (ppw * h)
    delta = torch.zeros((), dtype=torch.float64, device=DEV)
    for a, na in enumerate(n):
        i = torch.arange(na, device=DEV, dtype=torch.float64)
        da = torch.clamp(width - torch.minimum(i, na - 1 - i), min=0.0)
        delta = torch.maximum(delta, da.reshape([-1 if b == a else 1 for b in range(len(n))]))
    R = (2.0 * omega * (delta / width) ** 2).expand(n).contiguous()
    return c, R, omega, h, int(math.ceil(max(n) / ppw))


def _dense(n, seed):
    """A full complex vector, as the preconditioner meets in every iteration after the first."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.complex(torch.randn(n, generator=g, device=DEV, dtype=torch.float64),
                         torch.randn(n, generator=g, device=DEV, dtype=torch.float64))


def _point(n, seed, width):
    g = torch.Generator(device="cpu").manual_seed(seed)
    at = tuple(width + int(torch.randint(max(1, v - 2 * width), (1,), generator=g)) for v in n)
    F = torch.zeros(n, dtype=torch.complex128, device=DEV)
    F[tuple(min(a, v - 1) for a, v in zip(at, n))] = 1.0
    return F


def _batch_members(case, seed):
    """[(shape, width, seed, right-hand sides)]: one shared medium, then single uneven problems
    (their shapes follow from the case, their media from the seed)."""
    out = [(_shape(case), case["width"], seed, case["nrhs"])]
    g = torch.Generator(device="cpu").manual_seed(17 * case["n0"] + case["n1"])
    base = max(_shape(case))
    for i in range(case["fields"]):
        lo, hi = max(64, base // 4), base * 3 // 2
        n = tuple(int(v) for v in torch.randint(lo, hi + 1, (2,), generator=g))
        out.append((n, min(case["width"], min(n) // 4), seed + 100 + i, 1))
    return out


def _inputs(case, seed):
    """Everything the call needs, as tensors and numbers."""
    n = _shape(case)
    kind = case["kind"]
    if kind == "batch":
        members = []
        for shape, width, s, r in _batch_members(case, seed):
            members.append((_problem(shape, s, case["ppw"], width),
                            [_point(shape, s + 1000 + q, width) for q in range(r)]))
        return members
    p = _problem(n, seed, case["ppw"], case["width"], cmax=3.0 if kind == "gradient" else 4.5)
    if kind == "precond":
        return p, _dense(n, seed + 1)
    if kind == "solve":
        return p, _point(n, seed + 1, case["width"])
    F = torch.stack([_point(n, seed + 1 + q, case["width"]) for q in range(case["nrhs"])])
    W = _dense(tuple(F.shape), seed + 50)       # dL/dU of the misfit
    return p, F, W


# ---------------------------------------------------------------- the calls

def prepare(case, seed):
    kind, state = case["kind"], {"case": case}
    prec = tdp.F32 if case["prec"] == "f32" else tdp.F64
    kw = dict(prec=prec, steps_per_period=case["spp"], scheme=case["scheme"], damping=case["damping"])
    if kind == "batch":
        ops, nrhs, Fs, Ts = [], [], [], []
        for (c, R, omega, h, T), F in _inputs(case, seed):
            ops.append(tdp.Operator(c, R, omega, h, **kw))
            nrhs.append(len(F))
            Fs += F
            Ts.append(T)
        state.update(batch=tdp.Batch(ops, nrhs), F=Fs, T=Ts)
    elif kind == "gradient":
        (c, R, omega, h, T), F, W = _inputs(case, seed)
        state.update(m=(c ** -2.0).contiguous(), R=R, omega=omega, h=h, T=T, F=F, W=W)
    else:
        (c, R, omega, h, T), F = _inputs(case, seed)
        state.update(op=tdp.Operator(c, R, omega, h, **kw), F=F, T=T, out=torch.empty_like(F))
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "precond":
        return state["op"].precond(state["F"], state["T"], out=state["out"], variant=case["variant"])
    if kind == "solve":
        U, _ = state["op"].solve(state["F"], state["T"], fixed_iters=case["iters"])
        return U
    if kind == "batch":
        Us, _, _ = state["batch"].solve(state["F"], state["T"], fixed_iters=case["iters"])
        return Us
    m = state["m"].detach().requires_grad_(True)
    F = state["F"].detach().requires_grad_(True)
    U = autograd.helmholtz_solve(m, F, state["R"], state["omega"], state["h"], state["T"],
                                 steps_per_period=case["spp"])
    U.backward(state["W"])
    return {"U": U.detach(), "dm": m.grad, "dF": F.grad}


def _nodes(n):
    return float(math.prod(n))


def _steps(case, n, T):
    """Recurrence steps of one application; n_P from the bound on a medium of speed 1.5 and up."""
    S = TABLES[case["scheme"], len(n)][0]
    h = 1.0 / (max(n) + 1)
    wc2 = (2.0 * math.pi / (case["ppw"] * h)) ** 2
    lam = (_symbol_max(S, len(n)) / h ** 2) + wc2
    nmin = math.pi / math.asin(math.sqrt(wc2 / lam))
    return T * (4 * (int(nmin // 4) + 1) if case["spp"] == 0 else max(3, int(nmin) + 1))


def work(case):
    """Algorithmic work: the operator's node data (slowness, damping) and F read once and U
    written once per application, in the precision the fields have for the node data; flops of
    the stencil (two per point), the forcing and the u_{j-1} term per node and step."""
    word = 4 if case["prec"] == "f32" else 8
    n = _shape(case)
    per = {(2, "compact"): 24, (2, "fd2"): 16, (2, "q1"): 24, (3, "compact"): 44, (3, "fd2"): 20,
           (3, "q1"): 60}[len(n), case["scheme"]]
    if case["damping"] == "cell":
        per = 68
    elif case["variant"] == 1:
        per *= 2

    def app(shape, count):
        N = _nodes(shape)
        return (count * N * (32.0 + 2 * word),
                count * N * per * _steps(case, shape, math.ceil(max(shape) / case["ppw"])))

    kind = case["kind"]
    if kind == "precond":
        b, f = app(n, 1)
    elif kind == "solve":
        b, f = app(n, case["iters"] + 1)
    elif kind == "batch":
        b = f = 0.0
        for shape, _, _, r in _batch_members(case, 0):
            q = app(shape, r * (case["iters"] + 1))
            b, f = b + q[0], f + q[1]
    else:       # about a dozen applications per solve, a forward and an adjoint solve per source
        b, f = app(n, 24 * case["nrhs"])
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- the same in plain torch, 64 bits

def _esym(s, k):
    return sum(math.prod(s[a] for a in range(len(s)) if mask >> a & 1)
               for mask in range(1 << len(s)) if bin(mask).count("1") == k)


def _symbol_max(S, d):
    best = -math.inf
    for v in range(1 << d):
        s = [-1 if v >> a & 1 else 1 for a in range(d)]
        best = max(best, sum(S[k] * _esym(s, k) for k in range(d + 1)))
    return best * 2 ** d


def _cell_mean(v):
    """Mean over the corners of every cell, corners outside the grid taken at the nearest node."""
    for a in range(v.dim()):
        first, last = v.narrow(a, 0, 1), v.narrow(a, v.shape[a] - 1, 1)
        p = torch.cat([first, v, last], a)
        v = 0.5 * (p.narrow(a, 0, p.shape[a] - 1) + p.narrow(a, 1, p.shape[a] - 1))
    return v


def _offsets(d):
    out = [()]
    for _ in range(d):
        out = [o + (e,) for o in out for e in (-1, 0, 1)]
    return out


def _cell_weights(cells, n, o):
    """Sum of the cells that hold both a node and its neighbour at offset o, per node."""
    w = cells
    for a, e in enumerate(o):
        lo, hi = w.narrow(a, 0, n[a]), w.narrow(a, 1, n[a])
        w = lo if e < 0 else hi if e > 0 else lo + hi
    return w


class _Exact:
    """H, Table 1, Definition 4 and S_T^abd on one medium."""

    def __init__(self, case, p):
        c, R, self.omega, self.h, self.T = p
        self.n, d = tuple(c.shape), c.dim()
        S, M = TABLES[case["scheme"], d]
        cells = _cell_mean(c ** -2.0)
        self.cell = case["damping"] == "cell"
        wc = self.omega * math.sqrt(float(cells.max()))
        lam_s = _symbol_max(S, d) / self.h ** 2
        if self.cell:
            rcell = _cell_mean(R)
            lam_i = self.omega * float(rcell.max())
            nP = 4 if case["spp"] == 0 else 3
            while True:
                th = 2.0 * math.pi / nP
                al, be = th * th / (4 * math.sin(th / 2) ** 2), th / math.sin(th)
                w2 = wc * wc + be / th * (1 - math.cos(th)) * lam_i
                if th * th / al * (lam_s / w2 + 1) + th * be / al * (1 + math.cos(th)) * lam_i / w2 < 4:
                    break
                nP += 4 if case["spp"] == 0 else 1
            wc = math.sqrt(w2)
        else:
            nmin = math.pi / math.asin(wc / math.sqrt(lam_s + wc * wc))
            nP = 4 * (int(nmin // 4) + 1) if case["spp"] == 0 else max(3, int(nmin) + 1)
        self.nP = nP
        th = 2.0 * math.pi / nP
        dt = th / wc
        alpha, self.beta = th * th / (4 * math.sin(th / 2) ** 2), th / math.sin(th)
        self.g, self.cth = dt * dt / alpha, math.cos(th)
        self.H, self.B = [], []      # Re H and Im H (cell damping), per offset
        for o in _offsets(d):
            k = sum(1 for e in o if e)
            if S[k] == 0.0 and M[k] == 0.0:
                continue
            self.H.append((o, 2.0 ** (d - k) * S[k] / self.h ** 2
                           - self.omega ** 2 * M[k] * _cell_weights(cells, self.n, o)))
            if self.cell and M[k] != 0.0:
                self.B.append((o, self.omega * M[k] * _cell_weights(rcell, self.n, o)))
        # one step: u+ = A u - u- + g F, damped (Def. 2, Def. 6)
        self.A = [(o, -self.g * w) for o, w in self.H]
        for i, (o, w) in enumerate(self.A):
            if not any(o):
                self.A[i] = (o, w + 2.0 - self.g * wc * wc)
        lfac = self.beta * dt / (alpha * wc)
        self.R = self.omega * R
        self.half = 0.5 * lfac * self.R                  # l/2 of the node damping
        self.L = [(o, lfac * w) for o, w in self.B]

    def _pad(self, u):
        return torch.nn.functional.pad(u, (1, 1) * len(self.n))

    def _stencil(self, terms, up, out):
        for o, w in terms:
            v = up
            for a, e in enumerate(o):
                v = v.narrow(a, 1 + e, self.n[a])
            out.addcmul_(w, v)
        return out

    def apply_H(self, x):
        y = torch.zeros_like(x)
        self._stencil(self.H, self._pad(x), y)
        if self.cell:
            t = torch.zeros_like(x)
            return y + 1j * self._stencil(self.B, self._pad(x), t)
        return y + 1j * self.R * x

    def _window(self, s, rho):
        if s >= 1.0:
            return 0.0
        return 1.0 if s <= 1.0 - rho else math.sin(math.pi * (1.0 - s) / (2.0 * rho)) ** 2

    def precond(self, F, variant, rho=0.25):
        Ns = self.T * self.nP
        Fr, Fi = F.real.contiguous(), F.imag.contiguous()
        inner = (slice(1, -1),) * len(self.n)
        parts = 2 if (variant or self.cell) else 1
        size = tuple(v + 2 for v in self.n)
        lag = self.nP // 4 if self.nP % 4 == 0 else (self.nP + 2) // 4
        out = []
        for q in range(parts):
            up = torch.zeros(size, dtype=torch.float64, device=DEV)
            um = torch.zeros_like(up)
            snap = None
            for j in range(Ns):
                chi = self.g * self._window(1.0 - j / Ns, rho)
                ph = 2.0 * math.pi * j / self.nP
                a, b = chi * math.cos(ph), -chi * math.sin(ph)
                if q:
                    a, b = -b, a
                new = a * Fr
                new.add_(Fi, alpha=b)
                self._stencil(self.A, up, new)
                if self.cell:
                    self._stencil(self.L, um - self.cth * up, new)
                    new.sub_(um[inner])
                else:
                    new.sub_((1.0 - self.half) * um[inner])
                    new.div_(1.0 + self.half)
                um[inner] = new
                up, um = um, up
                if not q and j + 1 == Ns - lag:
                    snap = up[inner].clone()
            out.append(up[inner].clone())
        if parts == 2:
            return torch.complex(out[0], out[1])
        if self.nP % 4:
            phi = 2.0 * math.pi * lag / self.nP
            snap = (snap - math.cos(phi) * out[0]) / math.sin(phi)
        return torch.complex(out[0], snap)

    def gmres(self, F, iters, x=None, tol=None):
        """Left-preconditioned GMRES from x (default 0): `iters` iterations, or until the true
        residual is at most tol; the complex-linear map is used when a tolerance is asked for."""
        variant = 0 if tol is None else 1
        x = torch.zeros_like(F) if x is None else x
        while True:
            r = F - self.apply_H(x)
            if tol is not None and float(r.norm() / F.norm()) <= tol:
                return x
            z = self.precond(r, variant)
            beta = float(z.norm())
            V, Hm = [z / beta], torch.zeros((iters + 1, iters), dtype=torch.complex128)
            for i in range(iters):
                w = self.precond(self.apply_H(V[i]), variant)
                for _ in range(2):
                    for k, v in enumerate(V):
                        hk = torch.vdot(v.reshape(-1), w.reshape(-1))
                        w = w - hk * v
                        Hm[k, i] += hk.cpu()
                Hm[i + 1, i] = float(w.norm())
                V.append(w / Hm[i + 1, i].real.item())
            rhs = torch.zeros(iters + 1, dtype=torch.complex128)
            rhs[0] = beta
            y = torch.linalg.lstsq(Hm, rhs.reshape(-1, 1)).solution.reshape(-1)
            for k in range(iters):
                x = x + complex(y[k]) * V[k]
            if tol is None:
                return x

    def grad_m(self, case, lam, U):
        """omega^2 Re sum over corner pairs of a cell of M conj(lam) U, taken to the nodes."""
        d = len(self.n)
        M = TABLES[case["scheme"], d][1]
        lp, up = self._pad(lam), self._pad(U)
        corners = [tuple(v >> a & 1 for a in range(d)) for v in range(1 << d)]

        def at(p, e):
            for a in range(d):
                p = p.narrow(a, e[a], self.n[a] + 1)
            return p

        cell = torch.zeros([v + 1 for v in self.n], dtype=torch.float64, device=DEV)
        for b in corners:
            for g in corners:
                k = sum(x != y for x, y in zip(b, g))
                if M[k]:
                    cell += M[k] * (at(lp, b).conj() * at(up, g)).real
        cell *= self.omega ** 2
        for a in range(d):          # adjoint of the clamped corner mean
            N = self.n[a]
            out = 0.5 * (cell.narrow(a, 0, N) + cell.narrow(a, 1, N))
            out.narrow(a, 0, 1).add_(0.5 * cell.narrow(a, 0, 1))
            out.narrow(a, N - 1, 1).add_(0.5 * cell.narrow(a, N, 1))
            cell = out
        return cell


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = []
        for p, Fs in _inputs(case, seed):
            e = _Exact(case, p)
            out += [e.gmres(F, case["iters"]) for F in Fs]
        return out
    if kind == "gradient":
        p, F, W = _inputs(case, seed)
        e = _Exact(case, p)
        Us = [e.gmres(f, 10, tol=1e-12) for f in F]
        lams = [e.gmres(w.conj().resolve_conj(), 10, tol=1e-12).conj().resolve_conj() for w in W]
        dm = sum(e.grad_m(case, l, U) for l, U in zip(lams, Us))
        return {"U": torch.stack(Us), "dm": dm, "dF": torch.stack(lams)}
    p, F = _inputs(case, seed)
    e = _Exact(case, p)
    if kind == "solve":
        return e.gmres(F, case["iters"])
    return e.precond(F, case["variant"])
