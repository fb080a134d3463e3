"""The work that programs have this library do, as timed cases through its public entry points.

Every case works on a seeded synthetic problem of the kind the library is for: a wavespeed grid
c(x), a frequency given in grid points per wavelength (ppw) at the slowest wavespeed, an
absorbing layer, and right-hand sides that are point sources or complex Gaussian vectors.

`exact` gives the 64-bit result of a case in plain torch, written from the mathematics: the
7-point operator A = S - M - iD and its double-size and Fourier-spectral forms, the fixed-point
recursion of the shifted solves in the form the paper states it (Sec. 4.2, eq. fix-pt-exp), the
FCI step (Algorithm 1), and the U-Net with its gradients by autograd.
"""
import math

import numpy as np
import torch

from paper_1811_12378_amd import hfci


def listed():
    return [
        # one product of the smallest configuration (32^3, FP64): launch latency
        {"name": "apply_f64_32", "kind": "apply", "nz": 32, "ny": 32, "nx": 32, "prec": 64, "nvec": 1, "ppw": 10.0,
         "medium": "const", "im": 0.0},
        # products with a batch of Krylov vectors on an odd grid (residuals of a training harvest
        # are formed eight vectors at a time, in complex128)
        {"name": "apply_f64_odd", "kind": "apply", "nz": 131, "ny": 125, "nx": 119, "prec": 64, "nvec": 8,
         "ppw": 10.0, "medium": "grf", "im": 0.0},
        # the whole solver on the smallest configuration: constant c, point source, 8 poles,
        # degree 8, FP64, to 1e-8
        {"name": "solve_f64_32", "kind": "solve", "n": 32, "ppw": 10.0, "J": 8, "eps": 0.5, "q": 8, "tol": 1e-8},
        # the shifted solves of the plain FP64 method: 96^3 random medium, 12 poles, 4 sources
        # ("tune": the systems that the launch-shape tuner times, as programs that solve often
        # have it do once per operator; 0: the operator as it is created)
        {"name": "shifted_f64_96", "kind": "shifted", "form": "fd", "nz": 96, "ny": 96, "nx": 96, "prec": 64,
         "nrhs": 4, "ppw": 10.0, "medium": "grf", "rhs": "gauss", "J": 12, "eps": 0.25, "q": 8, "tune": 2},
        # the same problem in mixed precision, with the contour that the library's rule chooses
        # (eps 0.01, degree 10)
        {"name": "shifted_f32_96", "kind": "shifted", "form": "fd", "nz": 96, "ny": 96, "nx": 96, "prec": 32,
         "nrhs": 4, "ppw": 10.0, "medium": "grf", "rhs": "gauss", "J": 12, "eps": 0.01, "q": 10, "tune": 0},
        # the dominant work of the benchmark solve: 256^3 layered medium, 16 poles, point sources,
        # FP32 sweeps
        {"name": "shifted_f32_256", "kind": "shifted", "form": "fd", "nz": 256, "ny": 256, "nx": 256, "prec": 32,
         "nrhs": 4, "ppw": 8.0, "medium": "layered", "rhs": "point", "J": 16, "eps": 0.01, "q": 10, "tune": 8},
        # one application of the preconditioner in plain FP64 (the benchmark's FP64 arm), on a grid
        # whose sides differ
        {"name": "fci_f64_128", "kind": "fci", "nz": 112, "ny": 128, "nx": 144, "nrhs": 2, "ppw": 8.0,
         "medium": "layered", "rhs": "gauss", "J": 6, "eps": 0.04, "q": 10, "tune": 4},
        # independent operators of different sizes in one call, FP32
        {"name": "batch_f32", "kind": "batch", "count": 8, "lo": 48, "hi": 128, "prec": 32, "J": 8, "eps": 0.02,
         "q": 10},
        # the double-size formulation of the same shifted solves
        {"name": "two_f32_128", "kind": "shifted", "form": "two", "nz": 128, "ny": 128, "nx": 128, "prec": 32,
         "nrhs": 1, "ppw": 8.0, "medium": "layered", "rhs": "point", "J": 16, "eps": 0.02, "q": 8, "tune": 0},
        # the Fourier-spectral operator at its sampling of 2.25 points per wavelength
        {"name": "spectral_f32_128", "kind": "shifted", "form": "spectral", "nz": 128, "ny": 128, "nx": 128,
         "prec": 32, "nrhs": 1, "ppw": 2.25, "medium": "layered", "rhs": "point", "J": 16, "eps": 0.25, "q": 5,
         "tune": 0},
        # the learned preconditioner's network on a full grid, as one inner step evaluates it
        {"name": "net_eval_256", "kind": "net_eval", "nz": 256, "ny": 256, "nx": 256},
        # loss and gradients of one training crop with the residual loss
        {"name": "net_train_64", "kind": "net_train", "n": 64, "loss": 2},
    ]


def _side(rng, lo, hi):
    """A grid side, spread over its logarithm, odd ones among them."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("apply", "apply", "solve", "shifted", "shifted", "shifted", "shifted", "fci", "batch", "net_eval",
                       "net_train"))
    medium = rng.choice(("grf", "layered"))
    if kind == "apply":
        d = [_side(rng, 16, 256) for _ in range(3)]
        prec = rng.choice((32, 64))
        top = max(1, min(16, int(1.6e8 / (d[0] * d[1] * d[2]))))
        return {"kind": kind, "nz": d[0], "ny": d[1], "nx": d[2], "prec": prec, "nvec": rng.randint(1, top),
                "ppw": rng.uniform(6.0, 12.0), "medium": medium, "im": rng.choice((0.0, 0.4, -1.3))}
    if kind == "solve":
        return {"kind": kind, "n": rng.randint(16, 36), "ppw": rng.uniform(8.0, 12.0), "J": rng.choice((4, 6, 8, 10)),
                "eps": rng.uniform(0.2, 0.5), "q": rng.choice((4, 6, 7, 8)), "tol": rng.choice((1e-6, 1e-8))}
    if kind == "shifted":
        form = rng.choice(("fd", "fd", "fd", "two", "spectral"))
        prec = rng.choice((32, 32, 64))
        top = {"fd": 224, "two": 112, "spectral": 96}[form]
        d = [_side(rng, 24, top) for _ in range(3)]
        J = 2 * rng.randint(2, 8)
        nrhs = rng.randint(1, max(1, min(8, int(2.4e8 / (J * d[0] * d[1] * d[2])))))
        return {"kind": kind, "form": form, "nz": d[0], "ny": d[1], "nx": d[2], "prec": prec, "nrhs": nrhs,
                "ppw": rng.uniform(2.25, 4.0) if form == "spectral" else rng.uniform(6.0, 12.0), "medium": medium,
                "rhs": rng.choice(("point", "gauss")), "J": J, "eps": math.exp(rng.uniform(math.log(0.02), math.log(0.5))),
                "q": rng.choice((5, 8, 8, 10, 10, 12)), "tune": rng.choice((0, 2, 8)) if form == "fd" else 0}
    if kind == "fci":
        d = [_side(rng, 24, 144) for _ in range(3)]
        return {"kind": kind, "nz": d[0], "ny": d[1], "nx": d[2], "nrhs": rng.randint(1, 3), "ppw": rng.uniform(6.0, 12.0),
                "medium": medium, "rhs": rng.choice(("point", "gauss")), "J": 2 * rng.randint(2, 6),
                "eps": math.exp(rng.uniform(math.log(0.05), math.log(0.5))), "q": rng.choice((7, 8, 10)),
                "tune": rng.choice((0, 2))}
    if kind == "batch":
        lo = rng.choice((24, 32, 48))
        return {"kind": kind, "count": rng.randint(2, 10), "lo": lo, "hi": rng.randint(64, 120), "prec": rng.choice((32, 32, 64)),
                "J": rng.choice((4, 6, 8)), "eps": math.exp(rng.uniform(math.log(0.02), math.log(0.3))), "q": rng.choice((7, 8, 10))}
    if kind == "net_eval":
        d = [4 * _side(rng, 6, 64) for _ in range(3)]
        return {"kind": kind, "nz": d[0], "ny": d[1], "nx": d[2]}
    return {"kind": kind, "n": rng.choice([m for m in range(32, 100, 4) if m != 64]), "loss": rng.randint(0, 2)}


# ---- inputs -------------------------------------------------------------------------------

DAMP_CELLS, RHO2 = 8, 1.0
_ctx = None


def _context():
    """A program's one context: it owns the workspace that every call shares."""
    global _ctx
    if _ctx is None:
        _ctx = hfci.Context(0)
    return _ctx


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7fffffffffff)


def _grf(shape, gen):
    """Unit-variance Gaussian random field with correlation length 0.1."""
    w = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64)
    k = [torch.fft.fftfreq(m, d=1.0 / m, device="cuda", dtype=torch.float64) * 2 * math.pi for m in shape]
    k2 = k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2][None, None, :] ** 2
    g = torch.fft.ifftn(torch.fft.fftn(w) * torch.exp(-0.5 * k2 * 0.01)).real
    g = g - g.mean()
    return g / g.std()


def _medium(case, shape, gen):
    kind = case.get("medium", "grf")
    if kind == "const":
        return torch.ones(shape, device="cuda", dtype=torch.float64)
    g = _grf(shape, gen)
    if kind == "grf":
        return (2.5 + g).clamp(1.0, 4.5)
    v = 1.5 + 3.0 * torch.rand(8, generator=gen, device="cuda", dtype=torch.float64)
    layer = (torch.arange(shape[0], device="cuda") * 8 // shape[0]).clamp(max=7)
    return (v[layer][:, None, None] * (1.0 + 0.1 * g)).clamp(1.0, 5.0)


def _cells(shape):
    return min(DAMP_CELLS, min(shape) // 4)


def _problem(case, shape, seed):
    """(c, h, omega) of a case: h = 1 / (largest side)."""
    c = _medium(case, shape, _gen(seed)).contiguous()
    h = 1.0 / max(shape)
    return c, h, 2.0 * math.pi * float(c.min()) / (case["ppw"] * h)


def _vectors(case, count, shape, prec, seed, cells):
    dt = torch.complex128 if prec == 64 else torch.complex64
    gen = _gen(seed + 7919)
    if case.get("rhs", "gauss") == "gauss":
        return torch.randn((count,) + tuple(shape), generator=gen, device="cuda", dtype=torch.complex128).to(dt)
    f = torch.zeros((count,) + tuple(shape), device="cuda", dtype=dt)
    r = np.random.default_rng(seed + 17)
    for k in range(count):
        f[(k,) + tuple(int(r.integers(min(cells + 1, s // 2), max(s - cells - 1, s // 2 + 1))) for s in shape)] = 1.0
    return f


def _box(shape, s_h2, kappa, rho2):
    lo = sum(2.0 * (1.0 - math.cos(math.pi / (m + 1))) for m in shape)
    hi = sum(2.0 * (1.0 + math.cos(math.pi / (m + 1))) for m in shape)
    return s_h2 * lo - float(kappa.max()), s_h2 * hi - float(kappa.min()), rho2


def _poles(J, eps, rho2):
    phi = math.pi / J
    r = (rho2 / 2 + eps) / math.sin(phi)
    th = (2 * np.arange(1, J + 1) - 1) * phi
    return r * (np.cos(th) - math.cos(phi)) + 1j * (r * np.sin(th) - rho2 / 2), r * np.exp(1j * th) / J


def _ptilde(lam, z0, delta, q):
    x = -1j * delta * (lam - z0)
    term, total = np.ones_like(x), np.ones_like(x)
    for j in range(1, q + 1):
        term = term * x / j
        total = total + term
    return total


def _deltas(z, box, q):
    """Per pole the delta with the smallest bound on the fixed-point iteration's rate, and that
    rate (Sec. 4.2, eq. fix-pt-conv), on a scan that a program makes once per contour."""
    b1, b2, rho2 = box
    t = np.linspace(0.0, 1.0, 257)
    edge = np.concatenate([b1 + (b2 - b1) * t, b1 + (b2 - b1) * t - 1j * rho2, b1 - 1j * rho2 * t, b2 - 1j * rho2 * t])
    out, rates = [], []
    for zj in z:
        z0 = 0.5 * (b1 + b2) + 1j * zj.imag
        d = np.sign(zj.imag) * np.geomspace(0.02, 8.0, 160)
        nu = np.abs(_ptilde(edge[None, :], z0, d[:, None], q)).max(1) / np.abs(_ptilde(np.full((1, 1), zj), z0, d[:, None], q))[:, 0]
        k = int(np.argmin(nu))
        out.append(float(d[k]))
        rates.append(float(nu[k]))
    return out, rates


def _parts(case, shape, seed):
    """The scalars and diagonals of the normalised operator and the box of its form."""
    c, h, omega = _problem(case, shape, seed)
    cmin = float(c.min())
    s = cmin * cmin / (omega * omega)
    kappa = (cmin / c) ** 2
    cells = _cells(shape)
    dep = [(cells - torch.minimum(torch.arange(m, device="cuda"), m - 1 - torch.arange(m, device="cuda"))).clamp(min=0)
           for m in shape]
    depth = torch.maximum(torch.maximum(dep[0][:, None, None], dep[1][None, :, None]), dep[2][None, None, :])
    damp = RHO2 * (depth.double() / cells) ** 2
    box = _box(shape, s / h ** 2, kappa, RHO2)
    form, lam = case.get("form", "fd"), None
    if form == "two":
        R = RHO2 / 2 + math.sqrt(RHO2 ** 2 / 4 + box[1] + 1.0)
        box = (-1.0 - R, -1.0 + R, RHO2)
    elif form == "spectral":
        lam = torch.zeros(shape, device="cuda", dtype=torch.float64)
        for ax, m in enumerate(shape):
            i = torch.arange(m, device="cuda", dtype=torch.float64)
            k = 2 * math.pi * torch.minimum(i, m - i) / (m * h)
            lam += (k ** 2).reshape([m if a == ax else 1 for a in range(3)])
        lam *= s
        box = (-float(kappa.max()), float(lam.max()) - float(kappa.min()), RHO2)
    return {"c": c, "h": h, "omega": omega, "s": s, "sh2": s / h ** 2, "kappa": kappa, "damp": damp, "box": box, "lam": lam,
            "cells": cells, "form": form}


def _operator(case, shape, seed):
    p = _parts(case, shape, seed)
    cls = hfci.SpectralOperator if p["form"] == "spectral" else hfci.Operator
    op = cls(_context(), p["c"], p["h"], p["omega"], p["cells"], RHO2)
    if case.get("tune"):
        op.autotune(case.get("prec", 64), case["tune"])
    base = op
    if p["form"] == "two":
        op = base.case_two()
    return p, op


def _contour(case, p, op):
    z, _ = _poles(case["J"], case["eps"], RHO2)
    return hfci.Contour(op, case["J"], 1.0, case["eps"], case["q"], delta=_deltas(z, p["box"], case["q"])[0])


def _shape(case):
    return (case["nz"], case["ny"], case["nx"]) if "nz" in case else (case["n"],) * 3


def _shifted_rhs(case, p, seed):
    """The operator's right-hand sides: s f, or [0; s f] of the double-size form."""
    shape = _shape(case)
    f = _vectors(case, case["nrhs"], shape, case["prec"], seed, p["cells"]) * p["s"]
    return torch.stack([torch.zeros_like(f), f], 1).contiguous() if p["form"] == "two" else f


def _batch_cases(case):
    """The instances of an uneven batch: a side and a sampling each."""
    r = np.random.default_rng(1000 * case["lo"] + case["hi"])
    return [{"n": int(r.integers(case["lo"], case["hi"] + 1)), "ppw": float(r.uniform(6.0, 12.0)), "J": case["J"],
             "eps": case["eps"], "q": case["q"], "prec": case["prec"], "nrhs": 1} for _ in range(case["count"])]


LAYERS = ((16, 16), (16, 16), (16, 32), (32, 32), (32, 64), (64, 64), (96, 32), (32, 32), (48, 16), (16, 16))


def _net_params(seed):
    """He-normal kernels [27][cout][cin] and small biases layer by layer, then the head; the
    first layer's padded input channels are zero."""
    r = np.random.default_rng(seed)
    out = []
    for k, (cin, cout) in enumerate(LAYERS):
        real = 3 if k == 0 else cin
        w = np.zeros((27, cout, cin))
        w[:, :, :real] = r.standard_normal((27, cout, real)) * math.sqrt(2.0 / (27 * real))
        out += [w.ravel(), 0.02 * r.standard_normal(cout)]
    return np.concatenate(out + [0.1 * r.standard_normal(32), 0.02 * r.standard_normal(2)]).astype(np.float32)


def _net_input(shape, seed):
    """(x16, v): the network's input channels (a residual over its rms, omega^2 h^2 / c^2) and
    that residual."""
    gen = _gen(seed)
    c = _medium({"medium": "grf"}, shape, gen)
    v = torch.stack([_grf(shape, gen), _grf(shape, gen)], -1) + 0.5 * torch.randn(tuple(shape) + (2,), generator=gen,
                                                                                device="cuda", dtype=torch.float64)
    v = v / v.square().sum(-1).mean().sqrt()
    x = torch.zeros(tuple(shape) + (16,), device="cuda", dtype=torch.bfloat16)
    x[..., :2] = v.to(torch.bfloat16)
    x[..., 2] = ((2 * math.pi / 10.0) ** 2 * (c.min() / c) ** 2).to(torch.bfloat16)
    return x, v.float().contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "apply":
        p, op = _operator(case, _shape(case), seed)
        return {"kind": kind, "op": op, "x": _vectors(case, case["nvec"], _shape(case), case["prec"], seed, p["cells"]),
                "shift": complex(-0.3 if case["im"] else 0.0, case["im"])}
    if kind == "solve":
        case = dict(case, medium="const")
        p, op = _operator(case, _shape(case), seed)
        f = _vectors(dict(case, rhs="point"), 1, _shape(case), 64, seed, p["cells"])
        return {"kind": kind, "op": op, "c": _contour(case, p, op), "f": f,
                "opts": hfci.default_opts(precision=64, tol=case["tol"], max_it=500)}
    if kind == "shifted":
        p, op = _operator(case, _shape(case), seed)
        return {"kind": kind, "op": op, "c": _contour(case, p, op), "f": _shifted_rhs(case, p, seed)}
    if kind == "fci":
        p, op = _operator(case, _shape(case), seed)
        return {"kind": kind, "op": op, "c": _contour(case, p, op),
                "f": _vectors(case, case["nrhs"], _shape(case), 64, seed, p["cells"]),
                "opts": hfci.default_opts(precision=64)}
    if kind == "batch":
        ops, cons, fs = [], [], []
        for k, inst in enumerate(_batch_cases(case)):
            p, op = _operator(inst, _shape(inst), seed + 31 * k)
            ops.append(op)
            cons.append(_contour(inst, p, op))
            fs.append(_vectors(inst, 1, _shape(inst), case["prec"], seed + 31 * k, p["cells"])[0].contiguous())
        return {"kind": kind, "ops": ops, "cons": cons, "fs": fs}
    net = hfci.Net(_context())
    net.set_params(_net_params(seed))
    x, v = _net_input(_shape(case), seed)
    return {"kind": kind, "net": net, "x": x, "v": v, "loss": case.get("loss", 0)}


def run(state):
    kind = state["kind"]
    if kind == "apply":
        return hfci.apply(state["op"], state["x"], state["shift"])
    if kind == "solve":
        u, st = hfci.solve(state["op"], state["c"], state["f"], opts=state["opts"])
        return {"u": u, "its": st["its"]}
    if kind == "shifted":
        return hfci.shifted_solve(state["op"], state["c"], state["f"])[0]
    if kind == "fci":
        return hfci.fci_apply(state["op"], state["c"], state["f"], state["opts"])[0]
    if kind == "batch":
        return hfci.shifted_solve_batch(state["ops"], state["cons"], state["fs"])[0]
    if kind == "net_eval":
        return state["net"].eval(state["x"])
    loss = state["net"].train_step(state["x"], state["v"], update=False, loss_kind=state["loss"])
    return {"loss": loss, "grads": state["net"].get_grads()}


# ---- the least work of a pass -------------------------------------------------------------

def _steps(case, box):
    """Expected fixed-point steps per pole to reduce a residual by five: half of what the rate's
    bound asks for, a fifth near the real axis (vectors are not concentrated on the worst
    eigenvalue)."""
    z, _ = _poles(case["J"], case["eps"], RHO2)
    part = min(0.5, max(0.2, 0.5 * (case["eps"] / 0.08) ** 0.4))
    return [max(1, math.ceil(part * math.log(5.0) / -math.log(min(nu, 0.9999)))) for nu in _deltas(z, box, case["q"])[1]]


def _nominal_box(case, shape):
    """The box for the medium's usual range of kappa."""
    sh2 = (case["ppw"] / (2 * math.pi)) ** 2
    form = case.get("form", "fd")
    b1, b2 = -1.0, 12.0 * sh2 - 0.1
    if form == "two":
        R = 0.5 + math.sqrt(0.25 + b2 + 1.0)
        b1, b2 = -1.0 - R, -1.0 + R
    elif form == "spectral":
        b2 = 3.0 * math.pi ** 2 * sh2 - 0.1
    return b1, b2, RHO2


def work(case):
    kind = case["kind"]
    if kind in ("net_eval", "net_train"):
        n = float(np.prod(_shape(case)))
        mac = sum(27 * (3 if k == 0 else ci) * co / (1, 1, 8, 8, 64, 64, 8, 8, 1, 1)[k] for k, (ci, co) in enumerate(LAYERS))
        fwd = 2.0 * n * (mac + 32)
        par = 4.0 * sum(27 * a * b + b for a, b in LAYERS)
        if kind == "net_eval":
            return {"bytes": n * (3 * 2 + 8) + par, "flops": fwd}
        return {"bytes": n * (3 * 2 + 8) + 2 * par, "flops": 3.0 * fwd}
    if kind == "batch":  # the mean of the instances' sizes and samplings
        side = 0.5 * (case["lo"] + case["hi"])
        inst = dict(case, kind="shifted", n=int(side), nrhs=1, ppw=9.0)
        w = work(inst)
        return {k: case["count"] * v for k, v in w.items()}
    shape = _shape(case)
    n = float(np.prod(shape))
    e = 16.0 if case.get("prec", 64) == 64 else 8.0
    prod = 22.0 * n  # 7-point product with a complex diagonal and the factor's multiply-add
    if kind == "apply":
        return {"bytes": n * (case["nvec"] * 2 * e + e / 2), "flops": case["nvec"] * prod}
    if case.get("form") == "spectral":
        prod = n * (10.0 * math.log2(n) + 14.0)
    blocks = 2.0 if case.get("form") == "two" else 1.0
    products = case["q"] * sum(_steps(case, _nominal_box(case, shape)))
    if kind == "solve":  # about 40 preconditioned Arnoldi steps
        return {"bytes": n * (2 * e + 8), "flops": 40 * products * prod}
    nr = case["nrhs"]
    if kind == "fci":
        return {"bytes": n * (nr * 2 * e + 8), "flops": nr * products * prod}
    return {"bytes": n * (blocks * nr * (1 + case["J"]) * e + e / 2), "flops": nr * products * prod * (1.5 if blocks > 1 else 1.0)}


# ---- 64-bit results in plain torch --------------------------------------------------------

def _stencil(x, sh2):
    """sh2 (6 x - the six neighbours) with zero ghosts, x [..., nz, ny, nx]."""
    y = (6.0 * sh2) * x
    for ax in (-3, -2, -1):
        m = x.shape[ax]
        y.narrow(ax, 1, m - 1).sub_(x.narrow(ax, 0, m - 1), alpha=sh2)
        y.narrow(ax, 0, m - 1).sub_(x.narrow(ax, 1, m - 1), alpha=sh2)
    return y


def _product(p, x, shift):
    """(A - shift) x, or (B - shift) x with B = iC - I of the double-size form."""
    kd = p["kappa"] + 1j * p["damp"]
    if p["form"] == "two":
        x1, x2 = x[0], x[1]
        return torch.stack([-(1.0 + shift) * x1 + 1j * x2,
                            -1j * (_stencil(x1, p["sh2"]) - (p["kappa"] - 1.0) * x1) - (1.0 + shift + 1j * p["damp"]) * x2])
    if p["form"] == "spectral":
        return torch.fft.ifftn(p["lam"] * torch.fft.fftn(x)) - (kd + shift) * x
    y = _stencil(x, p["sh2"])
    return y.addcmul_(kd + shift, x, value=-1)


def _fixed_point(p, f, z, delta, q, reduce=5.0, most=200):
    """eq. fix-pt-exp from y = 0 until ||f - (A - z) y|| <= ||f|| / reduce."""
    b1, b2, _ = p["box"]
    z0 = 0.5 * (b1 + b2) + 1j * z.imag
    a, beta = -1j * delta, -1j * delta * (z - z0)
    pz = complex(_ptilde(np.array(z), z0, delta, q))
    y = torch.zeros_like(f)
    stop = float(torch.linalg.vector_norm(f)) / reduce
    for _ in range(most):
        t = _product(p, y, z0)
        if float(torch.linalg.vector_norm(f - t + (z - z0) * y)) <= stop:
            break
        k = (t - f).mul_(a)
        y = y.add_(k)
        for j in range(2, q + 1):
            k = _product(p, k, z0).sub_(f, alpha=beta ** (j - 1) / math.factorial(j - 1)).mul_(a / j)
            y.add_(k)
        y.div_(pz)
    return y


def _exact_shifted(case, p, f):
    z, _ = _poles(case["J"], case["eps"], RHO2)
    d, _ = _deltas(z, p["box"], case["q"])
    return torch.stack([torch.stack([_fixed_point(p, fr, complex(zj), dj, case["q"]) for fr in f]) for zj, dj in zip(z, d)])


def _gmres(p, b, tol=1e-13, most=600):
    n = b.numel()
    V = torch.zeros((most + 1, n), device="cuda", dtype=torch.complex128)
    H = np.zeros((most + 1, most), dtype=complex)
    beta = float(torch.linalg.vector_norm(b))
    V[0] = b.reshape(-1) / beta
    for j in range(most):
        w = _product(p, V[j].reshape(b.shape), 0.0).reshape(-1)
        for _ in range(2):
            h = V[: j + 1].conj() @ w
            w = w - h @ V[: j + 1]
            H[: j + 1, j] += h.cpu().numpy()
        H[j + 1, j] = float(torch.linalg.vector_norm(w))
        V[j + 1] = w / H[j + 1, j].real
        if j % 10 == 9 or j + 1 == most:
            e = np.zeros(j + 2, dtype=complex)
            e[0] = beta
            y = np.linalg.lstsq(H[: j + 2, : j + 1], e, rcond=None)[0]
            if np.linalg.norm(e - H[: j + 2, : j + 1] @ y) <= tol * beta:
                break
    return (torch.from_numpy(y).cuda() @ V[: j + 1]).reshape(b.shape)


def _unflatten(flat):
    out, at = [], 0
    for cin, cout in LAYERS:
        m = 27 * cin * cout
        out.append((flat[at:at + m].reshape(27, cout, cin), flat[at + m:at + m + cout]))
        at += m + cout
    return out, flat[at:at + 32].reshape(2, 16), flat[at + 32:at + 34]


def _conv(x, wb):
    w, b = wb
    Z, Y, X, _ = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1, 1, 1))
    y = b.expand(Z, Y, X, b.numel())
    for t in range(27):
        dz, dy, dx = t // 9, t // 3 % 3, t % 3
        y = y + xp[dz:dz + Z, dy:dy + Y, dx:dx + X] @ w[t].T
    return torch.relu(y)


def _pool(x):
    Z, Y, X, C = x.shape
    return x.reshape(Z // 2, 2, Y // 2, 2, X // 2, 2, C).mean((1, 3, 5))


def _up(x):
    return x.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)


def _unet(flat, x):
    L, hw, hb = _unflatten(flat)
    e1 = _conv(_conv(x, L[0]), L[1])
    e2 = _conv(_conv(_pool(e1), L[2]), L[3])
    b3 = _conv(_conv(_pool(e2), L[4]), L[5])
    d2 = _conv(_conv(torch.cat([_up(b3), e2], -1), L[6]), L[7])
    d1 = _conv(_conv(torch.cat([_up(d2), e1], -1), L[8]), L[9])
    return d1 @ hw.T + hb


def _loss(kind, o, v, kch):
    if kind == 0:
        return (o - v).square().sum() / v.square().sum()
    if kind == 2:
        o = o.permute(3, 0, 1, 2)
        y = (6.0 - kch) * o
        for ax in (1, 2, 3):
            m = o.shape[ax]
            y = y - torch.nn.functional.pad(o.narrow(ax, 0, m - 1), [0, 0] * (3 - ax) + [1, 0])
            y = y - torch.nn.functional.pad(o.narrow(ax, 1, m - 1), [0, 0] * (3 - ax) + [0, 1])
        o = y.permute(1, 2, 3, 0)
    re, im = (o * v).sum(), (o[..., 0] * v[..., 1] - o[..., 1] * v[..., 0]).sum()
    return 1.0 - (re ** 2 + im ** 2) / (o.square().sum() * v.square().sum())


def exact(case, seed):
    kind = case["kind"]
    if kind in ("net_eval", "net_train"):
        x, v = _net_input(_shape(case), seed)
        x, v = x.double(), v.double()
        flat = torch.from_numpy(_net_params(seed)).cuda().double()
        # the library's network computes with bfloat16 kernels
        L, _, _ = _unflatten(flat)
        for w, _ in L:
            w.copy_(w.to(torch.bfloat16).double())
        if kind == "net_eval":
            with torch.no_grad():
                return _unet(flat, x)
        flat.requires_grad_(True)
        loss = _loss(case["loss"], _unet(flat, x), v, x[..., 2])
        loss.backward()
        return {"loss": loss.detach(), "grads": flat.grad}
    if kind == "batch":
        out = []
        for k, inst in enumerate(_batch_cases(case)):
            p = _parts(inst, _shape(inst), seed + 31 * k)
            f = _vectors(inst, 1, _shape(inst), case["prec"], seed + 31 * k, p["cells"]).to(torch.complex128)
            out.append(_exact_shifted(inst, p, f)[:, 0])
        return out
    if kind == "solve":
        case = dict(case, medium="const")
        p = _parts(case, _shape(case), seed)
        f = _vectors(dict(case, rhs="point"), 1, _shape(case), 64, seed, p["cells"])
        return {"u": _gmres(p, p["s"] * f[0])[None], "its": None}
    p = _parts(case, _shape(case), seed)
    if kind == "apply":
        x = _vectors(case, case["nvec"], _shape(case), case["prec"], seed, p["cells"]).to(torch.complex128)
        return _product(p, x, complex(-0.3 if case["im"] else 0.0, case["im"]))
    if kind == "shifted":
        return _exact_shifted(case, p, _shifted_rhs(case, p, seed).to(torch.complex128))
    f = _vectors(case, case["nrhs"], _shape(case), 64, seed, p["cells"])
    z, sigma = _poles(case["J"], case["eps"], RHO2)
    y = _exact_shifted(case, p, f)
    w = sum(complex(s / zj) * yj for s, zj, yj in zip(sigma, z, y))
    aw = _product(p, w, 0.0)
    d = (aw.conj() * f).flatten(1).sum(1) / aw.abs().square().flatten(1).sum(1)
    return d[:, None, None, None] * w
