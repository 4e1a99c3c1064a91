"""Timing cases of the library's public entry points (Grid, Batch, Corrector).

listed() names the cases, draw(rng) gives further ones of the same ranges,
prepare(case, seed) makes the inputs and the handles a program keeps, run(state)
is one pass, work(case) what the pass cannot do without, and exact(case, seed)
the same outputs in 64 bits by plain torch (dense sine products or library
FFTs, none of this repository's code).

A case's "kind" selects the call:
  step        Grid.step_out / step / step_variable of n_steps steps
  batch       Batch.step of independent 2D instances
  corr_run    Corrector.run: coarse step, network, indicator, n_steps times
  corr_grad   Corrector.grad: network forward and backward of a batch of pairs
"""
import math
import os

import numpy as np
import torch

PROBLEMS = ("ac", "mms", "ex51", "ex52", "ex53")
EPS52 = 0.05  # Example 5.2
TH53, THC53 = 0.8, 1.6  # Example 5.3
CHANNELS = 32
TAU_C = 0.016  # coarse step of the learned corrector


def _step(name, problem, N, dtype, stages, steps, variable=False):
    N = list(N) + [0] * (3 - len(N))
    case = {"kind": "step", "problem": problem, "nx": N[0], "ny": N[1], "nz": N[2], "dtype": dtype, "stages": stages,
            "steps": steps, "variable": variable}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest grid of the tests and the smoke run: launches and latency only
        _step("ac2d_64_f64", "ac", (64, 64), "f64", 2, 100),
        # the benchmark: 3D Allen-Cahn, 255^3 unknowns, single precision
        _step("ac3d_256_f32", "ac", (256, 256, 256), "f32", 2, 10),
        # the same problem in the paper's precision
        _step("ac3d_256_f64", "ac", (256, 256, 256), "f64", 2, 10),
        # an ordinary 3D grid whose sizes are no powers of two, step sizes that vary
        _step("ac3d_ragged_f32_var", "ac", (240, 150, 100), "f32", 2, 10, True),
        # the paper's timing table (Example 5.1), its largest grid
        _step("ex51_4096x2048_f64", "ex51", (4096, 2048), "f64", 2, 10),
        # Example 5.2 on the grid of the paper's temporal rows: boundary data as part of f
        _step("ex52_1024x64x64_f64", "ex52", (1024, 64, 64), "f64", 2, 8),
        # Example 5.3: periodic grid, logarithmic reaction, the energy read at a checkpoint
        _step("ex53_128_f64", "ex53", (128, 128, 128), "f64", 2, 32),
        # the third-order scheme on the benchmark grid
        _step("three_256_f32", "ac", (256, 256, 256), "f32", 3, 5),
        # one Euler step at a time on a middle-sized 2D grid (calls from a user's own time loop)
        _step("ac2d_512x384_f32_one", "ac", (512, 384), "f32", 1, 1),
        # many independent 2D problems at once
        {"name": "batch_512", "kind": "batch", "count": 512, "dtype": "f32", "stages": 2, "steps": 5},
        # the trained corrector in a time loop
        {"name": "corr_run_512", "kind": "corr_run", "n": 512, "steps": 10},
        # one training batch of the corrector (the trainer's batch size)
        {"name": "corr_grad_512_b4", "kind": "corr_grad", "n": 512, "batch": 4},
    ]


def _size(rng, lo, hi):
    """An axis length: mostly products of 2, 3, 5 and 7 (what grids are made of), sometimes with factors up to 31
    (longer prime factors cost more than any listed case)."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    primes = (2, 3, 5, 7) if rng.random() > 0.12 else (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31)
    return min((m for m in range(lo, hi + 1) if _is_smooth(m, primes)), key=lambda m: (abs(m - n), m))


def _is_smooth(m, primes):
    for p in primes:
        while m % p == 0:
            m //= p
    return m == 1


def _pow2(rng, lo, hi):
    return 1 << rng.randint(lo, hi)


def draw(rng):
    kind = rng.choice(["ac1d", "ac2d", "ac2d", "ac2d_pow2", "ac3d", "ac3d", "ac3d_pow2", "mms", "ex51", "ex52", "ex53",
                       "batch", "corr_run", "corr_grad"])
    dtype = rng.choice(["f32", "f64"])
    stages = rng.choice([1, 2, 2, 3])
    variable = rng.random() < 0.25
    steps = rng.choice([1, 3, 8])
    if kind == "ac1d":
        return _step(None, "ac", (_size(rng, 16, 4096),), dtype, stages, 10 * steps, variable)
    if kind == "ac2d":
        return _step(None, "ac", (_size(rng, 16, 1536), _size(rng, 16, 1536)), dtype, stages, steps, variable)
    if kind == "ac2d_pow2":
        return _step(None, "ac", (_pow2(rng, 5, 11), _pow2(rng, 5, 11)), dtype, stages, steps, variable)
    if kind == "ac3d":
        return _step(None, "ac", tuple(_size(rng, 12, 216) for _ in range(3)), dtype, stages, steps, variable)
    if kind == "ac3d_pow2":
        return _step(None, "ac", tuple(rng.choice([64, 96, 128, 192, 256]) for _ in range(3)), dtype, stages, steps,
                     variable)
    if kind == "mms":
        return _step(None, "mms", (_size(rng, 64, 2048), _size(rng, 64, 2048)), dtype, stages, steps)
    if kind == "ex51":
        n = _pow2(rng, 6, 11)
        return _step(None, "ex51", (2 * n, n), dtype, stages, steps)
    if kind == "ex52":
        m = rng.choice([4, 8, 16, 24, 32, 48, 64])
        return _step(None, "ex52", (_size(rng, 64, 1024), m, m), dtype, stages, steps)
    if kind == "ex53":
        n = rng.choice([32, 48, 64, 96, 100, 128])
        return _step(None, "ex53", (n, n, n), dtype, stages, steps)
    if kind == "batch":
        return {"kind": "batch", "count": _size(rng, 8, 300), "dtype": dtype, "stages": rng.choice([1, 2]),
                "steps": steps}
    n = rng.choice([_size(rng, 64, 512), 256, 384])
    if kind == "corr_run":
        return {"kind": "corr_run", "n": n, "steps": rng.choice([2, 5, 10])}
    return {"kind": "corr_grad", "n": n, "batch": rng.randint(1, 4)}


# ----------------------------------------------------------------------------
# inputs


def _lengths(case):
    return [case[k] for k in ("nx", "ny", "nz") if case.get(k)]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _setup(case):
    """(intervals, mesh widths, D, tau, t0) of a step case."""
    N, p = _lengths(case), case["problem"]
    if p == "ac":
        return N, [1.0 / n for n in N], 0.02 ** 2, 0.005, 0.0
    if p == "mms":
        return N, [1.0 / n for n in N], 1.0, 2.0 ** -10, 0.0
    if p == "ex51":
        return N, [2.0 / N[0], 1.0 / N[1]], 0.5, 1.0 / 50, 0.0
    if p == "ex52":
        h = [math.sqrt(2.0) / N[0]] + [0.125 / n for n in N[1:]]
        return N, h, 1.0, 3.0 * math.sqrt(2.0) * EPS52 / 5.0 / 128, 0.0
    return N, [1.0 / n for n in N], 1e-4, 5.0 / 512, 0.0


def _axis(N, h, a=0.0):
    return a + h * torch.arange(1, N, dtype=torch.float64, device="cuda")


def _outer(vs):
    """Product over the axes, the first axis fastest."""
    out = torch.ones((), dtype=torch.float64, device="cuda")
    for v in reversed(vs):
        out = out.unsqueeze(-1) * v
    return out


def _wave(x, t):
    s, w = 3.0 / (math.sqrt(2.0) * EPS52), 2.0 * math.sqrt(2.0) * EPS52
    th = torch.tanh((x - s * t) / w)
    return 0.5 * (1.0 - th), 0.5 * s / w * (1.0 - th * th)


def _torch_dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _initial(case, seed):
    """The nodal values a pass starts from, in the case's dtype (first axis fastest)."""
    N, h, _, _, _ = _setup(case)
    p, g = case["problem"], _gen(seed)
    if p in ("ac", "ex53"):  # one random value per node
        shape = [n if p == "ex53" else n - 1 for n in reversed(N)]
        u = torch.rand(shape, dtype=torch.float64, device="cuda", generator=g) * 1.8 - 0.9
    else:  # the closed-form start, slightly disturbed so that every seed differs
        if p == "ex52":
            shape = [n - 1 for n in reversed(N)]
            u = _wave(_axis(N[0], h[0]), 0.0)[0].expand(shape).contiguous()
        else:
            u = _outer([torch.sin(math.pi * _axis(n, hh, 0.5 if (p == "ex51" and a == 0) else 0.0))
                        for a, (n, hh) in enumerate(zip(N, h))])
        u = u * (1.0 + 1e-3 * torch.rand(u.shape, dtype=torch.float64, device="cuda", generator=g))
    return u.to(_torch_dtype(case)).contiguous()


def _taus(case, seed):
    if not case["variable"]:
        return None
    rng = np.random.default_rng([int(seed), 7])
    return [0.005 * (1.0 + 0.5 * float(v)) for v in rng.uniform(-1.0, 1.0, case["steps"])]


def _batch_instances(case, seed):
    """(intervals, eps) per instance: the sizes are the case's, the diffusion the seed's."""
    Ns = np.random.default_rng([case["count"], 3]).choice([128, 192, 256, 384, 512], size=case["count"])
    eps = np.random.default_rng([int(seed), 11]).uniform(0.01, 0.05, case["count"])
    return [(int(n), float(e)) for n, e in zip(Ns, eps)]


def _states_2d(n_int, count, seed, t_end=1.0):
    """Coarsened Allen-Cahn states (float64) from random data: what the corrector meets after the transient."""
    u = torch.rand((count, n_int - 1, n_int - 1), dtype=torch.float64, device="cuda", generator=_gen(seed)) * 1.8 - 0.9
    return _Spectral([n_int, n_int], [1.0 / n_int] * 2, 4e-4).run(u, lambda t, v: v - v ** 3, [t_end / 40] * 40, 2)


def _pairs(case, seed):
    n = case["n"]
    un = _states_2d(n, case["batch"], seed)
    sp, f = _Spectral([n, n], [1.0 / n] * 2, 4e-4), (lambda t, v: v - v ** 3)
    uc = sp.run(un, f, [TAU_C], 2)
    uf = sp.run(un, f, [TAU_C / 8] * 8, 2)
    return [v.to(torch.float32).contiguous() for v in (un, uc, uf)]


def _start_weights(seed):
    """The parameters a training starts from: He-normal weights, zero biases, a small output layer."""
    rng = np.random.default_rng([int(seed), 13])
    C = CHANNELS
    parts = [rng.normal(0, math.sqrt(2.0 / 18), 18 * C), np.zeros(C)]
    for _ in range(4):
        parts += [rng.normal(0, math.sqrt(2.0 / (9 * C)), 9 * C * C), np.zeros(C)]
    parts += [rng.normal(0, 0.1 * math.sqrt(1.0 / (9 * C)), 9 * C), np.zeros(1)]
    return np.concatenate(parts).astype(np.float32)


def _weights():
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2209_11922_amd", "weights",
                        "corrector_ac512.npz")
    z = np.load(path, allow_pickle=False)
    return z["params"].astype(np.float32), float(z["s_out"])


def prepare(case, seed):
    import paper_2209_11922_amd as eife
    st = {"case": case}
    if case["kind"] == "step":
        N, h, D, tau, t0 = _setup(case)
        p = case["problem"]
        g = eife.Grid(N, h, D, case["dtype"], bc=eife.BC_PERIODIC if p == "ex53" else eife.BC_DIRICHLET)
        if p == "ex51":
            g.set_origin([0.5, 0.0])
        if p == "ex52":
            g.set_forcing(EPS52)
        if p == "ex53":
            g.set_forcing(TH53, THC53)
        g.set_phi(tau, case["stages"])
        st.update(grid=g, t0=t0, taus=_taus(case, seed),
                  f={"ac": eife.F_ALLEN_CAHN, "mms": eife.F_MMS_U2, "ex51": eife.F_EX51, "ex52": eife.F_TRAVELING_WAVE,
                     "ex53": eife.F_FLORY_HUGGINS}[p])
        st["u"] = _initial(case, seed)
        st["out"] = torch.empty_like(st["u"])
    elif case["kind"] == "batch":
        inst = _batch_instances(case, seed)
        b = eife.Batch([(n, n, 1.0 / n, 1.0 / n, e * e) for n, e in inst], case["dtype"])
        b.set_phi(0.01, case["stages"])
        st["stream"] = torch.cuda.Stream()
        b.autotune(None, st["stream"])
        st["batch"] = b
        st["f"] = eife.F_ALLEN_CAHN
        st["u"] = _batch_initial(case, seed, b.size())
        torch.cuda.synchronize()
    else:
        n = case["n"]
        params, s_out = _weights()
        net = eife.Corrector(n - 1, n - 1, case.get("batch", 1))
        net.set_params(params if case["kind"] == "corr_run" else _start_weights(seed))
        net.set_scale(s_out)
        st["net"] = net
        if case["kind"] == "corr_run":
            st["grids"] = []
            for tau in (TAU_C, TAU_C / 8):
                g = eife.Grid([n, n], [1.0 / n] * 2, 4e-4, "f32")
                g.set_phi(tau, 2)
                st["grids"].append(g)
            st["u0"] = _states_2d(n, 1, seed)[0].to(torch.float32).contiguous()
            st["u"] = torch.empty_like(st["u0"])
        else:
            st["pairs"] = _pairs(case, seed)
    return st


def _batch_initial(case, seed, count):
    u = torch.rand(count, dtype=torch.float64, device="cuda", generator=_gen(seed)) * 1.8 - 0.9
    return u.to(_torch_dtype(case))


def run(st):
    case = st["case"]
    if case["kind"] == "step":
        g = st["grid"]
        if st["taus"] is not None:
            return g.step_variable(st["u"], st["taus"], st["f"], st["t0"])
        if case["problem"] == "ex53":
            u = g.step(st["u"], case["steps"], st["f"], st["t0"])
            return u, g.energy(u, st["f"])
        return g.step_out(st["u"], st["out"], case["steps"], st["f"], st["t0"])
    if case["kind"] == "batch":
        return st["batch"].step(st["u"], case["steps"], st["f"], 0.0, stream=st["stream"])
    if case["kind"] == "corr_run":
        st["u"].copy_(st["u0"])
        coarse, fine = st["grids"]
        # an indicator bound wide enough that no step is repeated
        falls = st["net"].run(coarse, fine, st["u"], 0.0, TAU_C, case["steps"], 8, 10.0)
        return st["u"], falls
    loss, grad = st["net"].grad(*st["pairs"])
    return loss, grad


# ----------------------------------------------------------------------------
# what a pass cannot do without


def _step_flops(N, steps, stages):
    dofs = math.prod(N)
    per_transform = sum(2.5 * math.log2(2 * n) for n in N)  # a real odd transform of one line, per node
    return dofs * steps * stages * (2 * per_transform + 20)


def work(case):
    if case["kind"] == "step":
        N = _lengths(case)
        return {"bytes": 2 * math.prod(N) * (4 if case["dtype"] == "f32" else 8),
                "flops": _step_flops(N, case["steps"], case["stages"])}
    if case["kind"] == "batch":
        sizes = [128, 192, 256, 384, 512]
        nodes = case["count"] * sum(n * n for n in sizes) / len(sizes)
        flops = case["count"] * sum(_step_flops([n, n], case["steps"], case["stages"]) for n in sizes) / len(sizes)
        return {"bytes": 2 * nodes * (4 if case["dtype"] == "f32" else 8), "flops": flops}
    n = case["n"]
    net = 2 * 9 * (2 * CHANNELS + 4 * CHANNELS * CHANNELS + CHANNELS) * n * n
    if case["kind"] == "corr_run":
        return {"bytes": 2 * 4 * n * n, "flops": case["steps"] * (net + _step_flops([n, n], 1, 2))}
    return {"bytes": 3 * 4 * n * n * case["batch"], "flops": 3 * net * case["batch"]}


# ----------------------------------------------------------------------------
# the same outputs in 64 bits, by plain torch


class _Spectral:
    """Q1 finite elements in the sine (or periodic Fourier) basis, exponential Runge-Kutta steps in float64."""

    def __init__(self, N, h, D, periodic=False):
        self.N, self.h, self.D, self.periodic = N, h, D, periodic
        lam, w, self.S = [], [], []
        for n, hh in zip(N, h):
            k = torch.arange(n if periodic else n - 1, dtype=torch.float64, device="cuda")
            t = 2 * math.pi * k / n if periodic else math.pi * (k + 1) / n
            s = torch.sin(0.5 * t) ** 2
            lam.append(12.0 * s / (hh * hh * (3.0 - 2.0 * s)))
            w.append(6.0 / (6.0 - 4.0 * s))
            if not periodic:
                j = torch.arange(1, n, device="cuda", dtype=torch.int64)
                m = torch.outer(j, j) % (2 * n)
                self.S.append(math.sqrt(2.0 / n) * torch.sin(math.pi * m.double() / n))
        d = len(N)
        self.Lam = sum(v.reshape([-1] + [1] * a) for a, v in enumerate(lam)) * D
        self.w = math.prod(v.reshape([-1] + [1] * a) for a, v in enumerate(w)) if d > 1 else w[0]
        if d > 1:
            self.w = w[0]
            for a in range(1, d):
                self.w = self.w * w[a].reshape([-1] + [1] * a)

    def fwd(self, u):
        d = len(self.N)
        if self.periodic:
            return torch.fft.fftn(u, dim=tuple(range(-d, 0)))
        for a in range(d):
            v = u.movedim(-1 - a, -1).contiguous()
            u = (v.reshape(-1, v.shape[-1]) @ self.S[a]).reshape(v.shape).movedim(-1, -1 - a)
        return u.contiguous()

    def inv(self, u):
        return torch.fft.ifftn(u, dim=tuple(range(-len(self.N), 0))).real if self.periodic else self.fwd(u)

    def phis(self, z):
        """phi_1, phi_2, phi_3 at z <= 0: series below |z| = 1, recursion above."""
        small = z.abs() < 1.0
        zs, zl = torch.where(small, z, torch.zeros_like(z)), torch.where(small, -torch.ones_like(z), z)
        out, r = [], torch.expm1(zl)
        for k in (1, 2, 3):
            series = torch.zeros_like(z)
            for m in range(24, -1, -1):
                series = series * zs + 1.0 / math.factorial(m + k)
            big = r / zl ** k
            r = r - zl ** k / math.factorial(k)
            out.append(torch.where(small, series, big))
        return out

    def run(self, u, f, taus, stages, t0=0.0):
        H, t, coef = self.fwd(u), t0, None
        for q, tau in enumerate(taus):
            if coef is None or taus[q] != taus[q - 1]:
                coef = self.coefficients(tau, stages)
            nodes = [0.0, 0.5 if stages == 2 else 1.0 / 3.0, 2.0 / 3.0]
            G = []
            for i in range(stages):
                v = H if i == 0 else coef["e"][i] * H
                for j in range(i):
                    v = v + coef["a"][i][j] * G[j]
                G.append(self.w * self.fwd(f(t + nodes[i] * tau, self.inv(v))))
            H = coef["e"][0] * H
            for j in range(stages):
                H = H + coef["b"][j] * G[j]
            t += tau
        return self.inv(H)

    def coefficients(self, tau, stages):
        z = -tau * self.Lam
        p1, p2, p3 = self.phis(z)
        e = {0: torch.exp(z)}
        if stages == 1:
            return {"e": e, "a": {}, "b": [tau * p1]}
        if stages == 2:
            c = 0.5
            e[1] = torch.exp(c * z)
            return {"e": e, "a": {1: [c * tau * self.phis(c * z)[0]]}, "b": [tau * (p1 - p2 / c), tau * p2 / c]}
        c, d = 1.0 / 3.0, 2.0 / 3.0
        e[1], e[2] = torch.exp(c * z), torch.exp(d * z)
        d1, d2, _ = self.phis(d * z)
        a32 = tau * d * d / c * d2
        return {"e": e, "a": {1: [c * tau * self.phis(c * z)[0]], 2: [d * tau * d1 - a32, a32]},
                "b": [tau * (2 * p3 - (c + d) * p2 + c * d * p1) / (c * d), tau * (2 * p3 - d * p2) / (c * (c - d)),
                      tau * (2 * p3 - c * p2) / (d * (d - c))]}


def _reaction(case):
    N, h, D, _, _ = _setup(case)
    p = case["problem"]
    if p == "ac":
        return lambda t, u: u - u ** 3
    if p == "ex53":
        return lambda t, u: 0.5 * TH53 * torch.log((1 - u) / (1 + u)) + THC53 * u
    if p == "ex52":
        return lambda t, u: (u - u ** 3) / EPS52 ** 2 + _boundary_load(N, h, D, t)
    s = _outer([torch.sin(math.pi * _axis(n, hh, 0.5 if (p == "ex51" and a == 0) else 0.0))
                for a, (n, hh) in enumerate(zip(N, h))])
    if p == "ex51":
        return lambda t, u: 0.5 * math.pi ** 2 * (math.exp(-math.pi ** 2 * t) * s - u)
    return lambda t, u: u * u + (len(N) * math.pi ** 2 * D - 1.0) * math.exp(-t) * s - math.exp(-2 * t) * s * s


def _boundary_load(N, h, D, t):
    """-(M_b g' + D K_b g) / prod(h) at the interior nodes, g the wave on the boundary nodes."""
    x = h[0] * torch.arange(N[0] + 1, dtype=torch.float64, device="cuda")
    g, gt = _wave(x, t)
    shape = [n + 1 for n in reversed(N)]
    mask = torch.ones(shape, dtype=torch.float64, device="cuda")
    mask[tuple(slice(1, -1) for _ in N)] = 0.0

    def line(v, a, c0, c1):
        ax = v.dim() - 1 - a
        n = v.shape[ax]
        return c0 * v.narrow(ax, 1, n - 2) + c1 * (v.narrow(ax, 0, n - 2) + v.narrow(ax, 2, n - 2))

    def apply(v, stiff):
        for a, hh in enumerate(h):
            v = line(v, a, 2.0 / (hh * hh), -1.0 / (hh * hh)) if a == stiff else line(v, a, 2.0 / 3.0, 1.0 / 6.0)
        return v

    out = -apply(mask * gt, -1)
    for a in range(len(N)):
        out = out - D * apply(mask * g, a)
    return out


def _energy53(u, h, D):
    """(D/2) u^T K u + prod(h) sum F(u) on the periodic grid."""
    def line(v, a, c0, c1):
        ax = v.dim() - 1 - a
        return c0 * v + c1 * (torch.roll(v, 1, ax) + torch.roll(v, -1, ax))

    grad = 0.0
    for a in range(len(h)):
        v = u
        for b, hh in enumerate(h):
            v = line(v, b, 2.0 / hh, -1.0 / hh) if b == a else line(v, b, 4 * hh / 6, hh / 6)
        grad = grad + float((u * v).sum())
    F = 0.5 * TH53 * ((1 + u) * torch.log1p(u) + (1 - u) * torch.log1p(-u)) - 0.5 * THC53 * u * u
    return 0.5 * D * grad + math.prod(h) * float(F.sum())


def _shift(v, dy, dx):
    """v[:, y + dy, x + dx, :] with zeros outside."""
    out = torch.zeros_like(v)
    ny, nx = v.shape[1], v.shape[2]
    ys, xs = slice(max(0, -dy), ny - max(0, dy)), slice(max(0, -dx), nx - max(0, dx))
    yt, xt = slice(max(0, dy), ny + min(0, dy)), slice(max(0, dx), nx + min(0, dx))
    out[:, ys, xs] = v[:, yt, xt]
    return out


def _network(p, un, uc):
    """(network output, RMS change) in float64; p is the parameter vector (differentiable)."""
    c = torch.sqrt(((uc - un) ** 2).mean(dim=(1, 2), keepdim=True)) + 1e-30
    v = torch.stack([uc, (uc - un) / c], dim=-1)
    o = 0
    for layer in range(6):
        cin, cout = (2 if layer == 0 else CHANNELS), (1 if layer == 5 else CHANNELS)
        w = p[o:o + 9 * cin * cout]
        w = w.reshape(9, cin, cout) if layer in (0, 5) else w.reshape(9, cout, cin).transpose(1, 2)
        o += 9 * cin * cout
        acc = p[o:o + cout].expand(v.shape[:3] + (cout,)).reshape(-1, cout)
        o += cout
        for t in range(9):
            acc = acc + _shift(v, t // 3 - 1, t % 3 - 1).reshape(-1, cin) @ w[t].contiguous()
        v = acc.reshape(un.shape + (cout,))
        if layer < 5:
            v = torch.relu(v)
    return v[..., 0], c


def exact(case, seed):
    if case["kind"] == "step":
        N, h, D, tau, t0 = _setup(case)
        u = _initial(case, seed).double()
        sp = _Spectral(N, h, D, case["problem"] == "ex53")
        u = sp.run(u, _reaction(case), _taus(case, seed) or [tau] * case["steps"], case["stages"], t0)
        return (u, _energy53(u, h, D)) if case["problem"] == "ex53" else u
    if case["kind"] == "batch":
        inst = _batch_instances(case, seed)
        u = _batch_initial(case, seed, sum((n - 1) ** 2 for n, _ in inst)).double()
        out, at = [], 0
        for n, e in inst:
            m = (n - 1) ** 2
            sp = _Spectral([n, n], [1.0 / n] * 2, e * e)
            v = u[at:at + m].reshape(n - 1, n - 1)
            out.append(sp.run(v, lambda t, x: x - x ** 3, [0.01] * case["steps"], case["stages"]).reshape(-1))
            at += m
        return torch.cat(out)
    params, s_out = _weights()
    p = torch.tensor(params if case["kind"] == "corr_run" else _start_weights(seed), dtype=torch.float64, device="cuda")
    if case["kind"] == "corr_run":
        n = case["n"]
        u = _states_2d(n, 1, seed).to(torch.float32).double()
        sp = _Spectral([n, n], [1.0 / n] * 2, 4e-4)
        for _ in range(case["steps"]):
            uc = sp.run(u, lambda t, v: v - v ** 3, [TAU_C], 2)
            o, c = _network(p, u, uc)
            u = uc + s_out * c * o
        return u[0], None
    un, uc, uf = [v.double() for v in _pairs(case, seed)]
    p.requires_grad_(True)
    o, c = _network(p, un, uc)
    loss = ((o - (uf - uc) / (s_out * c)) ** 2).mean()
    loss.backward()
    return float(loss.detach()), p.grad.cpu().numpy()
