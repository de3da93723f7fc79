"""The work that programs give this library, as measured cases.

Each case is one call (or one forward and backward pair) of a public entry
point on the problems of the paper that the library's benchmark and tests
run: the heat equation on periodic grids, the free Schroedinger equation, the
Gross-Pitaevskii Strang step, the harmonic oscillator in nodal Hermite space
with a time-dependent potential, the vortex reconnection problem on graded
grids, the Hermite transforms, the batched integrator and the exponential
midpoint rule.  ``listed`` names twelve of them, ``draw`` gives others of the
same ranges, ``prepare`` makes what a program holds before the call (context,
prepared operators, tuned tiles, the state on the GPU), ``run`` is the call,
``work`` what it cannot do without, and ``exact`` the same result from plain
torch and numpy in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

TUNE_MS = 60          # budget of the autotuner where a program uses it
SIZES = (32, 48, 64, 96, 128, 192)     # mode lengths of the batched workload


def listed():
    return [
        # latency: a small 2-D heat run, 20 steps in one call
        {"name": "heat2d_64_fp64", "kind": "expstep", "problem": "heat", "d": 2, "n1": 64, "n2": 64, "n3": 1,
         "prec": "fp64", "steps": 20, "tuned": False},
        # an ordinary small 3-D run whose state fits a cache
        {"name": "schroedinger3d_64_fp32", "kind": "expstep", "problem": "schroedinger", "d": 3, "n1": 64, "n2": 64,
         "n3": 64, "prec": "fp32", "steps": 20, "tuned": False},
        # the reference precision at the benchmark's size
        {"name": "free3d_256_fp64", "kind": "expstep", "problem": "schroedinger", "d": 3, "n1": 256, "n2": 256,
         "n3": 256, "prec": "fp64", "steps": 2, "tuned": True},
        # the benchmark's workload: Strang steps in split half precision
        {"name": "gpe3d_256_fp16x2", "kind": "gpe", "d": 3, "n1": 256, "n2": 256, "n3": 256, "prec": "fp16x2",
         "identity": False, "steps": 8, "tuned": True},
        # the trajectory-accurate form for long runs
        {"name": "gpe3d_256_bf16x3_identity", "kind": "gpe", "d": 3, "n1": 256, "n2": 256, "n3": 256,
         "prec": "bf16x3", "identity": True, "steps": 4, "tuned": True},
        # a middle-sized run in single precision with the built-in tiles
        {"name": "gpe3d_100_fp32", "kind": "gpe", "d": 3, "n1": 100, "n2": 100, "n3": 100, "prec": "fp32",
         "identity": False, "steps": 4, "tuned": False},
        # spectral run with operators that change every step
        {"name": "ho3d_128_fp16x2", "kind": "ho", "n": 128, "prec": "fp16x2", "steps": 10, "tuned": True},
        # the paper's vortex grids: odd mode lengths, unaligned fibres
        {"name": "vortex3d_81_fp64", "kind": "vortex", "n": 81, "prec": "fp64", "steps": 10, "tuned": False},
        {"name": "vortex3d_141_fp16x2", "kind": "vortex", "n": 141, "prec": "fp16x2", "steps": 10, "tuned": True},
        # forward and backward Hermite transforms: real operators on complex data
        {"name": "transform3d_128_fp32", "kind": "transform", "n": 128, "K": 128, "prec": "fp32"},
        # many uneven independent instances, one step each
        {"name": "batch48_fp32", "kind": "batch", "count": 48, "mix": 5, "odd": False, "prec": "fp32", "steps": 1},
        # time-dependent generator: one exponential on the device per step
        {"name": "magnus3d_128_fp64", "kind": "magnus", "n": 128, "prec": "fp64", "steps": 4},
    ]


def _length(rng, lo, hi):
    """A mode length, spread over its logarithm; multiples of 8, other even
    numbers and odd ones all occur."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.4:
        return int(min(hi, max(lo, 8 * round(n / 8))))
    return int(n)


def draw(rng):
    kind = rng.choice(("expstep", "expstep", "gpe", "gpe", "ho", "vortex", "transform", "batch", "magnus"))
    prec = rng.choice(("fp64", "fp32", "bf16x3", "fp16x2"))
    if kind == "expstep":
        problem = rng.choice(("heat", "schroedinger"))
        d = rng.choice((2, 3))
        hi = 320 if d == 2 else 224
        lens = [_length(rng, 16, hi) for _ in range(d)] + [1]
        return {"kind": kind, "problem": problem, "d": d, "n1": lens[0], "n2": lens[1], "n3": lens[2], "prec": prec,
                "steps": rng.randint(1, 20) if math.prod(lens) < 300000 else rng.randint(1, 2),
                "tuned": rng.random() < 0.4}
    if kind == "gpe":
        lens = [_length(rng, 24, 224) for _ in range(3)]
        return {"kind": kind, "d": 3, "n1": lens[0], "n2": lens[1], "n3": lens[2], "prec": prec,
                "identity": rng.random() < 0.3, "steps": rng.randint(1, 4), "tuned": rng.random() < 0.4}
    if kind == "ho":
        return {"kind": kind, "n": _length(rng, 24, 144), "prec": prec, "steps": rng.randint(2, 10),
                "tuned": rng.random() < 0.4}
    if kind == "vortex":
        return {"kind": kind, "n": _length(rng, 32, 150), "prec": prec, "steps": rng.randint(2, 10),
                "tuned": rng.random() < 0.4}
    if kind == "transform":
        n = _length(rng, 24, 160)
        return {"kind": kind, "n": n, "K": n if rng.random() < 0.5 else rng.randint(max(1, n // 2), n), "prec": prec}
    if kind == "batch":
        return {"kind": kind, "count": rng.randint(4, 60), "mix": rng.randint(6, 1000000), "odd": rng.random() < 0.5,
                "prec": rng.choice(("fp64", "fp32", "bf16x3")), "steps": rng.randint(1, 2)}
    return {"kind": kind, "n": _length(rng, 24, 144), "prec": prec, "steps": rng.randint(1, 4)}


# ------------------------------------------------------- shared problem data

GPE = {"a": -8.0, "b": 8.0, "beta": 100.0, "tau": 1e-3}
FREE = {"a": -10.0, "b": 10.0, "tau": 0.01}
HEAT_TAU = 1e-3
HO = {"t0": 0.0, "tau": 0.02, "eps": 0.1}
VORTEX_TAU = 0.1
MAGNUS_TAU = 0.02


def _lens(case):
    if "n1" in case:
        return [case["n1"], case["n2"], case["n3"]][:case["d"]]
    return [case["n"]] * 3


def _complex_type(prec):
    return torch.complex128 if prec == "fp64" else torch.complex64


def _real_type(prec):
    return torch.float64 if prec == "fp64" else torch.float32


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _noise(shape, g):
    return torch.complex(torch.randn(shape, dtype=torch.float64, device="cuda", generator=g),
                         torch.randn(shape, dtype=torch.float64, device="cuda", generator=g)) / math.sqrt(2.0)


def _interior(n, a, b):
    h = (b - a) / (n + 1)
    return a + h * np.arange(1, n + 1, dtype=np.float64), h


def _axis(x, k, d):
    """Values along mode k + 1 of a d-dimensional state (mode 1 is the last torch axis)."""
    shape = [1] * d
    shape[d - 1 - k] = len(x)
    return torch.as_tensor(x, device="cuda").reshape(shape)


def _graded(n):
    xi = np.linspace(-1.0, 1.0, n)
    return 20.0 * np.sinh(2.0 * xi) / math.sinh(2.0)


def _graded_widths(x):
    h = np.diff(x)
    return np.concatenate([[h[0] / 2], (h[:-1] + h[1:]) / 2, [h[-1] / 2]])


def _instances(case):
    """Dimensions and kind of the batch's instances."""
    r = np.random.default_rng(case["mix"])
    out = []
    for _ in range(case["count"]):
        d = int(r.integers(2, 4))
        dims = [int(SIZES[j]) for j in r.integers(0, len(SIZES), size=d)]
        if case["odd"]:                  # the last mode of an instance may have any length
            dims[-1] = max(16, dims[-1] - int(r.integers(0, 16)))
        out.append((bool(r.random() < 0.5), dims))
    return out


def _state(case, seed):
    """The initial state (a list for the batch), as the case's type."""
    g = _generator(seed)
    kind = case["kind"]
    if kind == "batch":
        ts = []
        for cplx, dims in _instances(case):
            shape = tuple(reversed(dims))
            dt = _complex_type(case["prec"]) if cplx else _real_type(case["prec"])
            ts.append(torch.randn(shape, dtype=dt, device="cuda", generator=g))
        return ts
    lens = _lens(case)
    d = len(lens)
    shape = tuple(reversed(lens))
    if kind == "expstep" and case["problem"] == "heat":
        return torch.rand(shape, dtype=torch.float64, device="cuda", generator=g).to(_real_type(case["prec"]))
    ct = _complex_type(case["prec"])
    if kind == "expstep":                # wave packet of width 1 with a random momentum
        k0 = torch.rand(d, dtype=torch.float64, device="cuda", generator=g) * 4.0 - 2.0
        psi = torch.ones((1,) * d, dtype=torch.complex128, device="cuda")
        cell = 1.0
        for k in range(d):
            x, h = _interior(lens[k], FREE["a"], FREE["b"])
            xk = _axis(x, k, d)
            psi = psi * torch.polar(torch.exp(-0.5 * xk * xk), k0[k] * xk)
            cell *= h
        psi = psi + 1e-3 * _noise(shape, g)
        return (psi / torch.sqrt(cell * psi.abs().square().sum())).to(ct)
    if kind == "gpe":                    # Thomas-Fermi profile in the trap
        mu = 0.5 * (15.0 * GPE["beta"] / (4.0 * math.pi)) ** 0.4
        r2, cell = 0.0, 1.0
        for k in range(d):
            x, h = _interior(lens[k], GPE["a"], GPE["b"])
            r2 = r2 + _axis(x * x, k, d)
            cell *= h
        psi = torch.sqrt(torch.clamp(mu - 0.5 * r2, min=0.0) / GPE["beta"]) + 1e-3 * _noise(shape, g)
        return (psi / torch.sqrt(cell * psi.abs().square().sum())).to(ct)
    if kind == "vortex":                 # vortex and anti-vortex in a background of density 1
        x = _graded(case["n"])
        w = _graded_widths(x)
        x1, x2 = _axis(x, 0, 3), _axis(x, 1, 3)
        u = torch.ones((1,) * 3, dtype=torch.complex128, device="cuda")
        for s in (1.0, -1.0):
            z = torch.complex((x1 - 2.0 * s).expand(1, case["n"], case["n"]).contiguous(),
                              (s * x2).expand(1, case["n"], case["n"]).contiguous())
            u = u * (z / torch.sqrt(z.abs().square() + 1.0))
        u = u + 1e-3 * _noise(shape, g)
        return (torch.sqrt(_axis(w, 0, 3) * _axis(w, 1, 3) * _axis(w, 2, 3)) * u).to(ct)
    # Hermite problems: a random state over the nodes, decaying like the basis functions
    x, _ = _hermite(case["n"])
    env = 1.0
    for k in range(3):
        env = env * _axis(np.exp(-0.25 * np.minimum(x * x, 100.0)), k, 3)
    return (env * _noise(shape, g)).to(ct)


# ------------------------------------------------------------------ prepare

def prepare(case, seed):
    import paper_2103_01691_amd as mm
    kind, prec = case["kind"], case["prec"]
    ctx = mm.Context(0)
    s = {"case": case, "ctx": ctx, "x": _state(case, seed)}
    ops = {}

    def op(n, make, **kw):
        if n not in ops:
            ops[n] = ctx.mm_op_prepare(make(n), prec, **kw)
        return ops[n]

    if kind == "expstep":
        if case["problem"] == "heat":
            make = lambda n: mm.expm(mm.fd2_matrix(n, 0.0, 1.0, "periodic"), HEAT_TAU).real.copy()
        else:
            make = lambda n: mm.schrodinger_fd_exponential(n, FREE["a"], FREE["b"], 0.0, FREE["tau"])
        s["E"] = [op(n, make) for n in _lens(case)]
    elif kind == "gpe":
        make = lambda n: mm.schrodinger_fd_exponential(n, GPE["a"], GPE["b"], 1.0, GPE["tau"])
        s["E"] = [op(n, make, identity_split=case["identity"]) for n in _lens(case)]
    elif kind == "vortex":
        M, w = mm.nonuniform_neumann_d2(_graded(case["n"]))
        s["E"] = [ctx.mm_op_prepare(mm.expm(M, 0.5j * VORTEX_TAU), prec)] * 3
        s["w"] = [w] * 3
    elif kind in ("ho", "transform"):
        n = case["n"]
        K = case.get("K", n)
        Phi, Psi = mm.hermite_matrices(n)
        s["F"] = [ctx.mm_op_prepare(Phi[:K].copy(), prec)] * 3
        s["B"] = [ctx.mm_op_prepare(Psi[:, :K].copy(), prec)] * 3
        s["nodes"] = [mm.hermite_nodes(n)[0]] * 3
        if kind == "transform":
            s["spec"] = torch.empty((K,) * 3, dtype=s["x"].dtype, device="cuda")
            s["back"] = torch.empty_like(s["x"])
        elif case["tuned"]:
            s["E"] = [ctx.mm_op_prepare(mm.hermite_ho_exponential(n, HO["tau"]), prec)] * 3
    elif kind == "batch":
        heat = lambda n: mm.expm(mm.fd2_matrix(n, 0.0, 1.0, "periodic"), HEAT_TAU).real.copy()
        free = lambda n: mm.schrodinger_fd_exponential(n, FREE["a"], FREE["b"], 0.0, 1e-3)
        s["E"] = []
        for cplx, dims in _instances(case):
            row = []
            for n in dims:
                if (cplx, n) not in ops:
                    ops[cplx, n] = ctx.mm_op_prepare(free(n) if cplx else heat(n), prec)
                row.append(ops[cplx, n])
            s["E"].append(row)
    else:                                # magnus: the third mode's generator depends on time
        n = case["n"]
        s["B"] = [mm.hermite_ho_generator(n)] * 3
        s["d"] = [None, None, mm.hermite_nodes(n)[0]]
        s["g"] = _magnus_coefficients(case)
    if case.get("tuned"):
        ctx.mm_autotune(s["x"], s["E"], TUNE_MS)
    return s


def _magnus_coefficients(case):
    g = np.zeros((case["steps"], 3), dtype=np.complex128)
    g[:, 2] = -1j * np.sin((np.arange(case["steps"]) + 0.5) * MAGNUS_TAU) ** 2
    return g


# ---------------------------------------------------------------------- run

def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "expstep":
        return ctx.mumode_expstep(s["x"], s["E"], case["steps"])
    if kind == "gpe":
        return ctx.gpe_strang_step(s["x"], s["E"], GPE["tau"], GPE["beta"], case["steps"])
    if kind == "ho":
        return ctx.ho_strang_step(s["x"], s["F"], s["B"], s["nodes"], HO["t0"], HO["tau"], HO["eps"], case["steps"])
    if kind == "vortex":
        return ctx.vortex_strang_step(s["x"], s["E"], s["w"], VORTEX_TAU, case["steps"])
    if kind == "transform":
        ctx.mumode_transform(s["spec"], s["x"], s["F"])
        ctx.mumode_transform(s["back"], s["spec"], s["B"])
        return [s["spec"], s["back"]]
    if kind == "batch":
        return ctx.mumode_expstep_batched(s["x"], s["E"], case["steps"])
    return ctx.mumode_magnus_step(s["x"], s["B"], s["d"], s["g"], MAGNUS_TAU, case["steps"], case["prec"])


# --------------------------------------------------------------------- work

def work(case):
    kind = case["kind"]
    es = 8 if case["prec"] == "fp64" else 4          # bytes of a real value
    if kind == "batch":
        nbytes = flops = 0.0
        seen = set()
        for cplx, dims in _instances(case):
            c = 2 if cplx else 1
            N = float(np.prod(dims))
            nbytes += 2 * N * c * es
            for n in dims:
                flops += case["steps"] * (8 if cplx else 2) * n * N
                if (cplx, n) not in seen:
                    seen.add((cplx, n))
                    nbytes += n * n * c * es
        return {"bytes": nbytes, "flops": flops}
    lens = _lens(case)
    N = float(np.prod(lens))
    real = kind == "expstep" and case["problem"] == "heat"
    c = 1 if real else 2
    if kind == "transform":
        n, K = case["n"], case["K"]
        sizes = [(n ** 3, K * n * n), (K * n * n, K * K * n), (K * K * n, K ** 3)]
        flops = 2 * sum(4.0 * n * out for _, out in sizes)          # a real operator on complex data, both ways
        return {"bytes": c * es * (2.0 * n ** 3 + 2.0 * K ** 3) + 2 * n * K * es, "flops": flops}
    flops = case["steps"] * sum((2.0 if real else 8.0) * n * N for n in lens)
    if kind == "magnus":
        flops += case["steps"] * 7 * 8.0 * case["n"] ** 3            # the polynomial of the exponential
    return {"bytes": 2 * N * c * es + sum(n * n * c * es for n in set(lens)), "flops": flops}


# -------------------------------------------------------------------- exact

def _mode(T, L, k):
    """T x_{k+1} L in 64 bits (mode 1 is the last torch axis)."""
    L = torch.as_tensor(np.ascontiguousarray(L), device="cuda")
    if T.is_complex() and not L.is_complex():
        L = L.to(torch.complex128)
    ax = T.dim() - 1 - k
    M = T.movedim(ax, 0).contiguous()
    out = torch.matmul(L.contiguous(), M.reshape(M.shape[0], -1))
    return out.reshape((L.shape[0],) + M.shape[1:]).movedim(0, ax).contiguous()


def _second_difference(n, a, b, periodic):
    h = (b - a) / (n if periodic else n + 1)
    D = -2.0 * np.eye(n) + np.eye(n, k=1) + np.eye(n, k=-1)
    if periodic:
        D[0, n - 1] += 1.0
        D[n - 1, 0] += 1.0
    return D / h ** 2


def _symmetric_exponential(M, c):
    """exp(c M) of a real symmetric M."""
    lam, V = np.linalg.eigh(M)
    return (V * np.exp(c * lam)) @ V.T


def _free(n, tau):
    return _symmetric_exponential(-0.5 * _second_difference(n, FREE["a"], FREE["b"], False), -1j * tau)


def _hermite(n):
    """Gauss-Hermite nodes and the orthonormal Hermite functions scaled by the
    square roots of the function weights: Q[k, l] = phi_k(X_l) sqrt(w_l) is
    orthogonal (the eigenvectors of the Jacobi matrix)."""
    b = np.sqrt(np.arange(1, n) / 2.0)
    X, Q = np.linalg.eigh(np.diag(b, 1) + np.diag(b, -1))
    X = 0.5 * (X - X[::-1])
    return X, Q


def _hermite_pair(n, K):
    """Forward Phi[k, l] = phi_k(X_l) w_l and backward Psi[l, k] = phi_k(X_l)."""
    X, _ = _hermite(n)
    phi = np.zeros((n, n))
    phi[0] = math.pi ** -0.25 * np.exp(-0.5 * X * X)
    if n > 1:
        phi[1] = math.sqrt(2.0) * X * phi[0]
    for k in range(1, n - 1):
        phi[k + 1] = math.sqrt(2.0 / (k + 1)) * X * phi[k] - math.sqrt(k / (k + 1.0)) * phi[k - 1]
    w = 1.0 / (n * phi[n - 1] ** 2)
    return X, phi[:K] * w, phi[:K].T.copy()


def exact(case, seed):
    kind = case["kind"]
    x = _state(case, seed)
    if kind == "batch":
        out = []
        for (cplx, dims), t in zip(_instances(case), x):
            t = t.to(torch.complex128 if cplx else torch.float64)
            for _ in range(case["steps"]):
                for k, n in enumerate(dims):
                    L = _free(n, 1e-3) if cplx else _symmetric_exponential(_second_difference(n, 0.0, 1.0, True), HEAT_TAU)
                    t = _mode(t, L, k)
            out.append(t)
        return out
    lens = _lens(case)
    x = x.to(torch.complex128 if x.is_complex() else torch.float64)
    if kind == "expstep":
        heat = case["problem"] == "heat"
        L = [_symmetric_exponential(_second_difference(n, 0.0, 1.0, True), HEAT_TAU) if heat else _free(n, FREE["tau"])
             for n in lens]
        for _ in range(case["steps"]):
            for k in range(len(lens)):
                x = _mode(x, L[k], k)
        return x
    if kind == "gpe":
        turn = lambda v, t: v * torch.polar(torch.ones((), dtype=torch.float64, device="cuda"),
                                            -t * GPE["beta"] * v.abs().square())
        L = []
        for n in lens:
            xs, _ = _interior(n, GPE["a"], GPE["b"])
            H = -0.5 * _second_difference(n, GPE["a"], GPE["b"], False) + 0.5 * np.diag(xs * xs)
            L.append(_symmetric_exponential(H, -1j * GPE["tau"]))
        for _ in range(case["steps"]):
            x = turn(x, 0.5 * GPE["tau"])
            for k in range(len(lens)):
                x = _mode(x, L[k], k)
            x = turn(x, 0.5 * GPE["tau"])
        return x
    if kind == "vortex":
        xs = _graded(case["n"])
        w, h = _graded_widths(xs), np.diff(xs)
        S = np.diag(1.0 / h, 1) + np.diag(1.0 / h, -1)
        S -= np.diag(S.sum(1))
        L = _symmetric_exponential(S / np.sqrt(np.outer(w, w)), 0.5j * VORTEX_TAU)
        iw = 1.0 / (_axis(w, 0, 3) * _axis(w, 1, 3) * _axis(w, 2, 3))
        turn = lambda v, t: v * torch.polar(torch.ones((), dtype=torch.float64, device="cuda"),
                                            0.5 * t * (1.0 - iw * v.abs().square()))
        for _ in range(case["steps"]):
            x = turn(x, 0.5 * VORTEX_TAU)
            for k in range(3):
                x = _mode(x, L, k)
            x = turn(x, 0.5 * VORTEX_TAU)
        return x
    n = case["n"]
    X, Phi, Psi = _hermite_pair(n, case.get("K", n))
    if kind == "transform":
        spec = x
        for k in range(3):
            spec = _mode(spec, Phi, k)
        back = spec
        for k in range(3):
            back = _mode(back, Psi, k)
        return [spec, back]
    if kind == "ho":
        L = (Psi * np.exp(-1j * HO["tau"] * (np.arange(n) + 0.5))) @ Phi
        r2 = _axis(X * X, 0, 3) + _axis(X * X, 1, 3) + _axis(X * X, 2, 3)
        one = torch.ones((), dtype=torch.float64, device="cuda")
        for j in range(case["steps"]):
            t = HO["t0"] + j * HO["tau"]
            th, t1 = t + 0.5 * HO["tau"], t + HO["tau"]
            x = x * torch.polar(one, -0.5 * HO["eps"] * (math.cos(t) - math.cos(th)) * r2)
            for k in range(3):
                x = _mode(x, L, k)
            x = x * torch.polar(one, -0.5 * HO["eps"] * (math.cos(th) - math.cos(t1)) * r2)
        return x
    B = (Psi * (-1j * (np.arange(n) + 0.5))) @ Phi
    g = _magnus_coefficients(case)
    fixed = torch.linalg.matrix_exp(torch.as_tensor(MAGNUS_TAU * B)).numpy()
    for j in range(case["steps"]):
        A = MAGNUS_TAU * (B + g[j, 2] * np.diag(X))
        for k, L in enumerate((fixed, fixed, torch.linalg.matrix_exp(torch.as_tensor(A)).numpy())):
            x = _mode(x, L, k)
    return x
