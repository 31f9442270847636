"""The work that is timed: calls of this package's public entry points at the sizes its users run.

A case names one entry point (``kind``) and its sizes and options:

* ``box``    one box solve u = S f (``Problem.box_solve``, or ``box_solve_noalloc``);
* ``apply``  one product A psi of the boundary operator (``Problem.apply``);
* ``solve``  one Neumann solve (``Problem.solve_neumann``);
* ``batch``  many 2D Neumann solves at once (``Batch.solve_neumann``);
* ``step``   a few bidomain time steps from a given state (``Bidomain.step``).

Problem handles (geometry, grid and coefficients, as a user's program sets them up once) are kept
for the life of the process; every array is made anew from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2104_05024_amd import kfbi as K
from paper_2104_05024_amd import workloads as W

DT = 0.01                       # time step of the bidomain cases (kappa = 2 / DT)
_HANDLES = {}


# ----------------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call: a scalar 2D box solve, bound by launches and latency
        {"name": "box2d_64_f64", "kind": "box", "dim": 2, "cells": 64, "shape": "circle", "nodes": 128, "ncomp": 1,
         "aniso": False, "dtype": "f64", "entry": "problem"},
        # a coupled 3D box solve in the reduced precision of the mixed solvers, at the middle size
        {"name": "box3d_128_pair_f32", "kind": "box", "dim": 3, "cells": 128, "shape": "ellipsoid", "nodes": 8192,
         "ncomp": 2, "aniso": False, "dtype": "f32", "entry": "problem"},
        # the largest dense box solve: the coupled pair at 256^3
        {"name": "box3d_256_pair_f64", "kind": "box", "dim": 3, "cells": 256, "shape": "shell", "nodes": 40960,
         "ncomp": 2, "aniso": False, "dtype": "f64", "entry": "problem"},
        # one product of a small 2D scalar problem (the inner loop of a 2D solve)
        {"name": "apply2d_star128_f64", "kind": "apply", "dim": 2, "cells": 128, "shape": "star", "nodes": 256,
         "ncomp": 1, "aniso": False, "dtype": "f64"},
        # one product of the paper's anisotropic 2D pair at a finer grid
        {"name": "apply2d_circle512_pair_f64", "kind": "apply", "dim": 2, "cells": 512, "shape": "spline_circle",
         "nodes": 511, "ncomp": 2, "aniso": True, "dtype": "f64"},
        # the product that dominates the flagship workload: thick shell, coupled pair, 256^3
        {"name": "apply3d_shell256_pair_f64", "kind": "apply", "dim": 3, "cells": 256, "shape": "shell",
         "nodes": 40960, "ncomp": 2, "aniso": False, "dtype": "f64"},
        # the scalar product in reduced precision (inner product of a mixed solve) at 256^3
        {"name": "apply3d_psphere256_f32", "kind": "apply", "dim": 3, "cells": 256, "shape": "psphere",
         "nodes": 32768, "ncomp": 1, "aniso": False, "dtype": "f32"},
        # a whole scalar 3D Neumann solve with inner products in FP32 and FP64 refinement
        {"name": "solve3d_ellipsoid128_mixed", "kind": "solve", "dim": 3, "cells": 128, "shape": "ellipsoid",
         "nodes": 8191, "ncomp": 1, "aniso": False, "precision": 1, "tol": 1e-10},
        # many uneven 2D problems (64..1024 cells) in lockstep
        {"name": "batch2d_64_mixed", "kind": "batch", "problems": 64, "sizes": "64,128,256,512,1024", "precision": 1,
         "tol": 1e-10},
        # steps of the paper's 2D example with its virtual electrode, potentials returned
        {"name": "step2d_circle128", "kind": "step", "dim": 2, "cells": 128, "shape": "spline_circle", "nodes": 128,
         "ncomp": 2, "aniso": True, "precision": 0, "warm": 0, "steps": 3, "tol": 1e-11, "stimulus": True},
        # steps of a small 3D tissue in mixed precision
        {"name": "step3d_ellipsoid64_mixed", "kind": "step", "dim": 3, "cells": 64, "shape": "ellipsoid",
         "nodes": 2049, "ncomp": 2, "aniso": False, "precision": 2, "warm": 0, "steps": 4, "tol": 1e-8,
         "stimulus": False},
        # the flagship: steps of the thick shell at 256^3, all FP64
        {"name": "step3d_shell256", "kind": "step", "dim": 3, "cells": 256, "shape": "shell", "nodes": 40960,
         "ncomp": 2, "aniso": False, "precision": 0, "warm": 0, "steps": 3, "tol": 1e-10, "stimulus": False},
    ]


def draw(rng):
    kind = rng.choice(["box", "box", "apply", "apply", "apply", "solve", "batch", "step"])
    if kind == "batch":
        top = rng.choice([128, 256, 512, 1024])
        return {"kind": "batch", "problems": rng.randint(3, 61),
                "sizes": ",".join(str(s) for s in (64, 128, 256, 512, 1024) if s <= top),
                "precision": rng.choice([0, 1]), "tol": 1e-10}
    dim = rng.choice([2, 3])
    ncomp = 2 if kind == "step" else rng.choice([1, 2])
    top = {2: 10, 3: 8}[dim] - (1 if kind == "step" else 0)
    cells = 2 ** rng.randint(5 if kind in ("solve", "step") else 4, top)
    if dim == 2:
        shape = rng.choice(["circle", "star", "spline_circle"]) if cells >= 64 else "circle"
        nodes = int(cells * rng.uniform(1.0, 2.2)) | 1
    else:
        shape = rng.choice(["ellipsoid", "psphere", "shell"]) if cells >= 64 else "sphere"
        nodes = int(cells * cells * rng.uniform(0.35, 0.65)) | 1
    c = {"kind": kind, "dim": dim, "cells": cells, "shape": shape, "nodes": nodes, "ncomp": ncomp,
         "aniso": rng.random() < 0.4}
    if kind in ("box", "apply"):
        c["dtype"] = rng.choice(["f64", "f32"])
    if kind == "box":
        c["entry"] = "noalloc" if cells <= (64 if dim == 3 else 512) and rng.random() < 0.3 else "problem"
    if kind == "solve":
        c.update(precision=rng.choice([0, 1]) if ncomp == 1 else 0, tol=1e-10)
    if kind == "step":
        c.update(precision=0, warm=0, steps=rng.randint(2, 4), tol=1e-11 if dim == 2 else 1e-10,
                 stimulus=rng.random() < 0.3)
        if dim == 3 and not c["aniso"] and not c["stimulus"]:
            # mixed precision or the projected start: looser solves, as they are used
            c.update(rng.choice([{}, {"precision": 2}, {"warm": 3}]), tol=1e-8)
    return c


# ----------------------------------------------------------------------------- handles

def _interface(case):
    n, s = case["nodes"], case["shape"]
    if s == "circle":
        return W.circle2d(0.6, n)
    if s == "star":
        return W.star2d(0.7, 0.15, 5, n)
    if s == "spline_circle":
        return W.spline_circle(0.8, n)
    if s == "sphere":
        return W.sphere(0.6, n)
    if s == "ellipsoid":
        return W.ellipsoid(n_nodes=n)
    if s == "psphere":
        return W.perturbed_sphere(n_nodes=n)
    return W.thick_shell(n_nodes=n)


def _coeffs(case):
    """sigma = 1 or (1, 2), or the ratios 30 : 5 and 20 : 10 along and across the fibres."""
    d = case["dim"]
    if case["ncomp"] == 1:
        return W.Coeffs(1, [[3.0] + [0.5] * (d - 1) if case["aniso"] else [1.0] * d], 400.0)
    if case["aniso"]:
        return W.Coeffs(2, [[3.0] + [0.5] * (d - 1), [2.0] + [1.0] * (d - 1)], 2.0 / DT)
    return W.bidomain_coeffs(d, W.BidomainParams(), DT)


def _problem(case):
    key = tuple(case[k] for k in ("dim", "cells", "shape", "nodes", "ncomp", "aniso"))
    if key not in _HANDLES:
        _HANDLES[key] = K.Problem(_interface(case), W.box(case["dim"], case["cells"]), _coeffs(case))
    return _HANDLES[key]


def _batch(case):
    key = (case["problems"], case["sizes"])
    if key not in _HANDLES:
        probs = W.batch_2d(case["problems"], 2, tuple(int(s) for s in case["sizes"].split(",")))
        _HANDLES[key] = (K.Batch(probs), [(gr.cells, co.kappa) for _, gr, co in probs])
    return _HANDLES[key]


# ----------------------------------------------------------------------------- inputs

def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.float64


def _waves(rng, dim, cells, count=4):
    """A smooth field on the (cells - 1)^dim interior nodes: a few products of sines and cosines
    of seeded frequencies and phases, of order one, as a flat float64 tensor."""
    x = torch.linspace(-1.2, 1.2, cells + 1, dtype=torch.float64, device="cuda")[1:-1]
    out = torch.zeros((cells - 1,) * dim, dtype=torch.float64, device="cuda")
    for _ in range(count):
        term = torch.full((1,) * dim, float(rng.uniform(0.2, 0.5)), dtype=torch.float64, device="cuda")
        for a in range(dim):
            shape = [1] * dim
            shape[a] = cells - 1
            term = term * torch.sin(float(rng.uniform(0.5, 3.0)) * x + float(rng.uniform(0, 6.28))).reshape(shape)
        out += term
    return out.reshape(-1)


def _noise(seed, shape, dtype):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    return torch.randn(shape, dtype=dtype, device="cuda", generator=g)


def _ball(case, centre, radius=0.25):
    x = torch.linspace(-1.2, 1.2, case["cells"] + 1, dtype=torch.float64, device="cuda")[1:-1]
    r2 = torch.zeros((1,) * case["dim"], dtype=torch.float64, device="cuda")
    for a in range(case["dim"]):               # axis 0 (x) is the last, fastest one
        shape = [1] * case["dim"]
        shape[case["dim"] - 1 - a] = case["cells"] - 1
        r2 = r2 + ((x - centre[a]) ** 2).reshape(shape)
    return (r2 < radius * radius).to(torch.float64).reshape(-1).contiguous()


def prepare(case, seed):
    rng = np.random.default_rng(int(seed))
    kind = case["kind"]
    if kind == "batch":
        b, probs = _batch(case)
        f = torch.cat([kap * _waves(rng, 2, cells) for cells, kap in probs])
        g = 0.5 * torch.sin(torch.linspace(0.0, float(rng.uniform(20, 60)), b.L, dtype=torch.float64, device="cuda"))
        return {"kind": kind, "batch": b, "f": f, "g": g, "opts": {"tol": case["tol"], "precision": case["precision"]}}
    dim, cells, nc = case["dim"], case["cells"], case["ncomp"]
    n = (cells - 1) ** dim
    s = {"kind": kind}
    if kind == "box":
        s["f"] = _noise(seed, (nc, n), _dtype(case))
        if case["entry"] == "noalloc":
            s["grid"], s["coeffs"] = W.box(dim, cells), _coeffs(case)
            return s
    s["problem"] = p = _problem(case)
    if kind == "apply":
        s["psi"] = _noise(seed, (nc, p.M), _dtype(case))
    elif kind == "solve":
        # a compatible pair: the source (kappa v, -kappa v) with insulated boundary; scalar: any data
        v = 200.0 * _waves(rng, dim, cells)
        s["f"] = torch.stack([v, -v]) if nc == 2 else v.reshape(1, -1)
        t = torch.linspace(0.0, float(rng.uniform(20, 60)), p.M, dtype=torch.float64, device="cuda")
        s["g"] = None if nc == 2 else 0.5 * torch.sin(t).reshape(1, -1)
        s["opts"] = {"tol": case["tol"], "precision": case["precision"]}
    elif kind == "step":
        fhn = W.BidomainParams()
        u = rng.normal(size=dim)
        c = 0.6 * u / np.linalg.norm(u)
        s["V0"] = _ball(case, c) + 0.02 * _waves(rng, dim, cells)
        s["q0"] = 0.01 * _waves(rng, dim, cells)
        s["V"], s["q"] = torch.empty_like(s["V0"]), torch.empty_like(s["q0"])
        s["hist"] = torch.zeros(2, 2, p.M, dtype=torch.float64, device="cuda")
        s["phi"] = s["stim"] = None
        if case["stimulus"]:
            # the paired electrode (anode and cathode of one radius), potentials wanted too
            left, right = [-0.3] + [0.0] * (dim - 1), [0.3] + [0.0] * (dim - 1)
            s["stim"] = float(rng.uniform(5, 15)) * (_ball(case, left) - _ball(case, right))
            s["phi"] = torch.zeros(2, n, dtype=torch.float64, device="cuda")
        s["stepper"] = K.Bidomain(p, fhn, tol=case["tol"], precision=case["precision"], warm_start=case["warm"],
                                  inner_tol=2e-3)
        s["steps"] = case["steps"]
    return s


def run(s):
    kind = s["kind"]
    if kind == "box":
        if "problem" in s:
            return s["problem"].box_solve(s["f"])
        return K.box_solve_noalloc(s["grid"], s["coeffs"], s["f"])
    if kind == "apply":
        return s["problem"].apply(s["psi"])
    if kind == "solve":
        u, psi, _ = s["problem"].solve_neumann(s["g"], s["f"], **s["opts"])
        return {"u": u} if s["g"] is None else {"u": u, "psi": psi}
    if kind == "batch":
        u, psi, _ = s["batch"].solve_neumann(s["g"], s["f"], **s["opts"])
        return {"u": u, "psi": psi}
    # a simulation started from a stored state and carried on for a few steps
    s["V"].copy_(s["V0"])
    s["q"].copy_(s["q0"])
    s["hist"].zero_()
    s["stepper"].reset()
    for _ in range(s["steps"]):
        s["stepper"].step(s["V"], s["q"], s["hist"], DT, phi=s["phi"], I_stim=s["stim"])
    out = {"V": s["V"], "q": s["q"]}
    if s["phi"] is not None:
        out["phi"] = s["phi"]
    return out


# ----------------------------------------------------------------------------- minimal work and exact values

def _box_work(dim, cells, ncomp, elem):
    """One field read and one written; the transforms of all axes but one, there and back
    (2.5 log2 M operations per value), and a constant-coefficient solve along the last."""
    n = ncomp * (cells - 1) ** dim
    return 2.0 * n * elem, n * (5.0 * (dim - 1) * math.log2(cells) + 12.0)


def _apply_work(dim, cells, ncomp, nodes, elem):
    """The density read and the result written; the stencil weights of about four grid-line
    crossings and of one fit per node, with their indices; the box solve between them, its field
    written and read once."""
    k = 10 if dim == 3 else 6
    b, f = _box_work(dim, cells, ncomp, elem)
    per_node = 5 * k * (4 + 8 * ncomp)
    return b + nodes * (per_node + 16.0 * ncomp), f + nodes * 10.0 * k * ncomp


def work(case):
    if case["kind"] == "box":
        b, f = _box_work(case["dim"], case["cells"], case["ncomp"], 4 if case["dtype"] == "f32" else 8)
    elif case["kind"] == "apply":
        b, f = _apply_work(case["dim"], case["cells"], case["ncomp"], case["nodes"], 4 if case["dtype"] == "f32" else 8)
    elif case["kind"] == "batch":
        b = f = 0.0
        sizes = [int(s) for s in case["sizes"].split(",")]
        for s in sizes:                        # a volume solve, a final solve and some five products each
            n = case["problems"] / len(sizes)
            bb, bf = _box_work(2, s, 1, 8)
            ab, af = _apply_work(2, s, 1, 2 * s, 4 if case["precision"] else 8)
            b, f = b + n * (2 * bb + 5 * ab), f + n * (2 * bf + 5 * af)
    else:
        bb, bf = _box_work(case["dim"], case["cells"], case["ncomp"], 8)
        ab, af = _apply_work(case["dim"], case["cells"], case["ncomp"], case["nodes"], 8 if case["precision"] == 0 else 4)
        b, f = 2 * bb + 5 * ab, 2 * bf + 5 * af
        if case["kind"] == "step":
            b, f = case["steps"] * b, case["steps"] * f
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """The box solve by dense sine matrices in 64 bits.  The other kinds rest on the geometry
    tables, which plain torch does not give."""
    if case["kind"] != "box":
        return None
    dim, cells, nc = case["dim"], case["cells"], case["ncomp"]
    n, grid, co = cells - 1, W.box(dim, cells), _coeffs(case)
    f = _noise(seed, (nc, n ** dim), _dtype(case)).to(torch.float64).reshape([nc] + [n] * dim)
    k = torch.arange(1, cells, dtype=torch.float64, device="cuda")
    kn = torch.remainder(torch.outer(k, k), 2 * cells)
    S = torch.sin(math.pi / cells * kn)
    lam = (2.0 / grid.h * torch.sin(0.5 * math.pi / cells * k)) ** 2

    def modes(v):
        for _ in range(dim):                   # transform the last axis, then bring the next one there
            v = torch.matmul(v, S).movedim(-1, 1).contiguous()
        return v

    f = modes(f)
    a = []
    for c in range(nc):
        s = torch.zeros([1] * dim, dtype=torch.float64, device="cuda")
        for ax in range(dim):
            shape = [1] * dim
            shape[dim - 1 - ax] = n
            s = s + co.D[c][ax] * lam.reshape(shape)
        a.append(s)
    scale = (2.0 / cells) ** dim
    if nc == 1:
        u = scale * f / (a[0] + co.kappa)
    else:
        det = a[0] * a[1] + co.kappa * (a[0] + a[1])
        u = torch.stack([scale * ((a[1] + co.kappa) * f[0] + co.kappa * f[1]) / det,
                         scale * (co.kappa * f[0] + (a[0] + co.kappa) * f[1]) / det])
    return modes(u).reshape(nc, -1)
