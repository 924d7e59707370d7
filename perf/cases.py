"""Timed cases of the library: filters, stencils, their Jacobi iteration and scans, called through the
binding as a program would call them, with buffers the program already holds.

The sizes are those of bench.py and workloads.py (8192 x 8192 images and 512^3 grids), the small and the
ragged sizes of the parity tests, and generic ones in between.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1907_06154_amd.binding as ssam

DTYPE = {"f32": torch.float32, "f64": torch.float64}
SIZE = {"f32": 4, "f64": 8}

MAX_GRID_BYTES = 1 << 30               # one buffer of the largest listed grids and arrays
MAX_FLOPS = 2 * 400 * 8192 * 8192      # the largest listed filter
MAX_SWEEP_BYTES = 10 * 2 * (1 << 30)   # the largest listed iteration: ten sweeps over 512^3 fp64


def listed():
    return [
        # a thumbnail or one tile of a larger picture: latency
        {"name": "conv2d_3x3_f32_512", "op": "conv2d", "W": 512, "H": 512, "M": 3, "N": 3, "dtype": "f32", "boundary": "clamp"},
        # the ordinary image filter on the benchmark's image
        {"name": "conv2d_5x5_f32_8192", "op": "conv2d", "W": 8192, "H": 8192, "M": 5, "N": 5, "dtype": "f32", "boundary": "clamp"},
        # the largest filter of the benchmark's sweep
        {"name": "conv2d_20x20_f32_8192", "op": "conv2d", "W": 8192, "H": 8192, "M": 20, "N": 20, "dtype": "f32", "boundary": "clamp"},
        # a camera picture whose rows have an odd length
        {"name": "conv2d_9x9_f32_4003x3001", "op": "conv2d", "W": 4003, "H": 3001, "M": 9, "N": 9, "dtype": "f32", "boundary": "clamp"},
        # Jacobi solver, double precision, large 2D domain
        {"name": "iterate2d_box1_f64_8192", "op": "iterate", "W": 8192, "H": 8192, "D": 1, "shape": "box", "r": 1, "steps": 16,
         "dtype": "f64", "boundary": "zero"},
        # diffusion on a small domain with a ghost layer: odd extents, few launches
        {"name": "iterate2d_star1_f32_1023x1025", "op": "iterate", "W": 1023, "H": 1025, "D": 1, "shape": "star", "r": 1, "steps": 10,
         "dtype": "f32", "boundary": "clamp"},
        # one time step of a high-order wave propagator (the rest of the step is the program's own)
        {"name": "stencil3d_star4_f32_512", "op": "stencil", "W": 512, "H": 512, "D": 512, "shape": "star", "r": 4, "dtype": "f32",
         "boundary": "zero"},
        # Jacobi solver, 7-point Laplacian, the benchmark's grid
        {"name": "iterate3d_star1_f64_512", "op": "iterate", "W": 512, "H": 512, "D": 512, "shape": "star", "r": 1, "steps": 10,
         "dtype": "f64", "boundary": "zero"},
        # the 27-point smoother on a medium grid with odd extents
        {"name": "iterate3d_box1_f64_201x203x199", "op": "iterate", "W": 201, "H": 203, "D": 199, "shape": "box", "r": 1, "steps": 4,
         "dtype": "f64", "boundary": "clamp"},
        # filter of a volume (tomography, microscopy)
        {"name": "conv3d_5x5x5_f32_512", "op": "conv3d", "W": 512, "H": 512, "D": 512, "M": 5, "N": 5, "K": 5, "dtype": "f32",
         "boundary": "clamp"},
        # prefix sums of an array far beyond the caches, and of a mid-sized one of odd length
        {"name": "scan_f32_268435456", "op": "scan", "n": 1 << 28, "dtype": "f32"},
        {"name": "scan_f64_1000003", "op": "scan", "n": 1000003, "dtype": "f64"},
    ]


def _extent(rng, lo, hi):
    """Log-uniform in lo .. hi; half of them as they fall (odd ones among them), half rounded to a multiple of 32."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        v = max(32, (v + 16) // 32 * 32)
    return min(max(v, lo), hi)


def _fits(case):
    w = work(case)
    if case["op"] == "scan":
        return case["n"] * SIZE[case["dtype"]] <= MAX_GRID_BYTES
    points = case["W"] * case["H"] * case.get("D", 1)
    return (points * SIZE[case["dtype"]] <= MAX_GRID_BYTES and w["flops"] <= MAX_FLOPS
            and w["bytes"] * case.get("steps", 1) <= MAX_SWEEP_BYTES)


def _draw(rng):
    op = rng.choices(["conv2d", "stencil2d", "iterate2d", "stencil3d", "iterate3d", "conv3d", "scan"],
                     weights=[30, 10, 15, 10, 10, 15, 10])[0]
    case = {"dtype": rng.choices(["f32", "f64"], weights=[2, 1])[0]}
    if op == "scan":
        case.update(op="scan", n=int(round(math.exp(rng.uniform(math.log(1000), math.log(1 << 28))))))
        return case
    case["boundary"] = rng.choice(["clamp", "zero"])
    if op in ("conv2d", "stencil2d", "iterate2d"):
        case.update(W=_extent(rng, 256, 8192), H=_extent(rng, 256, 8192))
    else:
        case.update(W=_extent(rng, 48, 512), H=_extent(rng, 48, 512), D=_extent(rng, 48, 512))
    if op == "conv2d":
        kind = rng.choices(["square", "rectangle", "wide"], weights=[60, 25, 15])[0]
        if kind == "square":
            case["M"] = case["N"] = rng.randint(2, 20)
        elif kind == "rectangle":
            case["M"], case["N"] = rng.randint(1, 20), rng.randint(1, 20)
        else:
            case["M"] = case["N"] = rng.randint(21, 32)
        case["op"] = "conv2d"
    elif op == "conv3d":
        if rng.random() < 0.6:
            case["M"] = case["N"] = case["K"] = rng.randint(2, 7)
        else:
            case["M"], case["N"], case["K"] = (rng.randint(1, 9) for _ in range(3))
        case["op"] = "conv3d"
    else:
        flat = op.endswith("2d")
        case["shape"] = rng.choice(["star", "box"] if flat else ["star", "box", "faces_edges"])
        most = {"star": 6 if flat else 4, "box": 4 if flat else 2, "faces_edges": 1}[case["shape"]]
        case["r"] = rng.randint(1, most)
        if flat:
            case["D"] = 1
        case["op"] = "stencil" if op.startswith("stencil") else "iterate"
        if case["op"] == "iterate":
            case["steps"] = int(round(math.exp(rng.uniform(math.log(2), math.log(24 if flat else 10)))))
    return case


def draw(rng):
    while True:
        case = _draw(rng)
        if _fits(case):
            return case


def _taps(case):
    """The filter or coefficient box as a boolean mask, [n][m] or [k][n][m]."""
    if case["op"] == "conv2d":
        return np.ones((case["N"], case["M"]), dtype=bool)
    if case["op"] == "conv3d":
        return np.ones((case["K"], case["N"], case["M"]), dtype=bool)
    r, dims = case["r"], 2 if case["D"] == 1 else 3
    off = np.indices((2 * r + 1,) * dims) != r
    budget = {"star": 1, "faces_edges": 2, "box": dims}[case["shape"]]
    return off.sum(axis=0) <= budget


def _grid_shape(case):
    return (case["H"], case["W"]) if case.get("D", 1) == 1 and case["op"] != "conv3d" else (case["D"], case["H"], case["W"])


def _weights(case, seed):
    """Filters: uniform in [-1, 1).  Stencils: non-negative with sum 1, as a diffusion step has."""
    rng = np.random.default_rng(seed)
    mask = _taps(case)
    if case["op"] in ("conv2d", "conv3d"):
        w = rng.uniform(-1.0, 1.0, mask.shape)
    else:
        w = np.where(mask, rng.uniform(0.0, 1.0, mask.shape), 0.0)
        w /= w.sum()
    return w.astype(np.float32 if case["dtype"] == "f32" else np.float64)


def _field(case, seed):
    """Pictures and volumes: uniform in [0, 1).  Solver fields and scanned arrays: uniform in [-1, 1)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = (case["n"],) if case["op"] == "scan" else _grid_shape(case)
    x = torch.rand(shape, generator=g, device="cuda", dtype=DTYPE[case["dtype"]])
    return x if case["op"].startswith("conv") else x.mul_(2.0).sub_(1.0)


def prepare(case, seed):
    x = _field(case, seed)
    state = {"op": case["op"], "x": x, "y": torch.empty_like(x)}
    if case["op"] == "scan":
        need = ssam.ssam_scan_workspace_bytes(case["n"], x.dtype)
        state["work"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    else:
        state.update(w=_weights(case, seed), boundary=case["boundary"], steps=case.get("steps", 1))
    return state


def run(state):
    op, x, y = state["op"], state["x"], state["y"]
    if op == "conv2d":
        return ssam.ssam_conv2d(x, state["w"], boundary=state["boundary"], d_out=y)
    if op == "conv3d":
        return ssam.ssam_conv3d(x, state["w"], boundary=state["boundary"], d_out=y)
    if op == "stencil":
        f = ssam.ssam_stencil2d if x.dim() == 2 else ssam.ssam_stencil3d
        return f(x, state["w"], boundary=state["boundary"], d_out=y)
    if op == "iterate":
        result = ssam.ssam_stencil_iterate(x, y, state["w"], state["steps"], boundary=state["boundary"])
        if result is y:        # the solver goes on from the field it has reached
            state["x"], state["y"] = y, x
        return result
    return ssam.ssam_scan(x, d_out=y, d_work=state["work"])


def work(case):
    if case["op"] == "scan":
        return {"bytes": 2 * case["n"] * SIZE[case["dtype"]], "flops": case["n"]}
    points = case["W"] * case["H"] * case.get("D", 1)
    taps = int(_taps(case).sum())
    return {"bytes": 2 * points * SIZE[case["dtype"]], "flops": 2 * taps * points * case.get("steps", 1)}


def tolerance(case):
    """About four times the distance from exact(): measured up to 3.1e-7 (fp32, 400 taps) and 3.3e-16 (fp64
    scan); filters of up to 1024 taps and other orders of the sums leave a little more."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 2e-15, "max": 2e-14}


def _sweep(x, w, anchor, clamp):
    """out[p] = sum_k w[k] x[p + k - anchor] in 64 bits, a tap at a time."""
    pad = []
    for size, a in zip(reversed(w.shape), reversed(anchor)):
        pad += [a, size - 1 - a]
    xp = torch.nn.functional.pad(x[None, None], pad, mode="replicate" if clamp else "constant")[0, 0]
    out = torch.zeros_like(x)
    for at in np.argwhere(w != 0.0):
        view = xp[tuple(slice(int(o), int(o) + n) for o, n in zip(at, x.shape))]
        out.add_(view, alpha=float(w[tuple(at)]))
    return out


def exact(case, seed):
    x = _field(case, seed).double()
    if case["op"] == "scan":
        return torch.cumsum(x, 0)
    w = _weights(case, seed).astype(np.float64)
    anchor = [s // 2 for s in w.shape]
    for _ in range(case.get("steps", 1)):
        x = _sweep(x, w, anchor, case["boundary"] == "clamp")
    return x
