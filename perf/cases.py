"""The hologram work that users of this package have it do, as timed cases.

Every case is one pass through the public entry points of ``binding``:

  op         forward    I = forward(...)
             noalloc    I = forward_noalloc(..., out=I), the serving-loop call
             step       (I, G) = forward_residual(..., T), then backward(..., G)
             backward   gradients for a given G = dL/dI
             autograd   CGHFunction, L = 0.5 ||I - T||^2, L.backward()
             f64        forward_f64
  variant    the phase arithmetic (ignored by f64)
  cloud      how the points are drawn: "uniform" in the aperture, or on a
             "mesh" surface (z over [0.2, 1.5] m)

The sizes are those of ``workloads.WORKLOADS``, of the N-sweep at 1920 x 1024
and of the ragged parity tests.  Points are uniform clouds (or a height-field
surface) as in ``workloads``; the target T is the hologram of a hidden cloud
and the trainable cloud is that cloud perturbed, as when fitting.
"""
import math

import numpy as np
import torch

from paper_1002_0916_amd import binding as cgh

PITCH, WAVELENGTH = 8e-6, 633e-9


def _case(name, op, variant, nx, ny, n, zlo, zhi, cloud="uniform"):
    c = {"op": op, "variant": variant, "nx": nx, "ny": ny, "n": n, "zlo": zlo, "zhi": zhi,
         "cloud": cloud}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A small display refreshed in a serving loop without allocation: the
        # smallest call, where latency and launches count.
        _case("serve_256", "noalloc", "compensated", 256, 256, 64, 0.3, 0.6),
        # A ragged crop (no side a multiple of a tile) with an odd point count,
        # as fitted interactively.
        _case("ragged_step_333", "step", "compensated", 333, 197, 700, 0.3, 0.6),
        # The paper's shape: one hologram by the plain FP32 phase ...
        _case("paper_forward_plain", "forward", "plain", 1920, 1024, 1024, 0.5, 1.0),
        # ... the default fitting step (hologram, residual, gradients) ...
        _case("paper_step", "step", "compensated", 1920, 1024, 1024, 0.5, 1.0),
        # ... the same by the 16-bit hi/lo contraction ...
        _case("paper_step_f16x3", "step", "separable_f16x3", 1920, 1024, 1024, 0.5, 1.0),
        # ... and by the paper's recurrence (Eq. (2)).
        _case("paper_step_recurrence", "step", "recurrence", 1920, 1024, 1024, 0.5, 1.0),
        # The FP64 reference hologram that the FP32 variants are judged by.
        _case("paper_forward_f64", "f64", "compensated", 1920, 1024, 1024, 0.5, 1.0),
        # A full-HD hologram of a mesh object, at full precision and in the
        # single-plane fp16 format of the precision study.
        _case("mesh8k_forward", "forward", "compensated", 1920, 1080, 8192, 0.2, 1.5, "mesh"),
        _case("mesh8k_forward_f16", "forward", "separable_f16", 1920, 1080, 8192, 0.2, 1.5,
              "mesh"),
        # Gradients alone for an upstream G from the caller's own loss.
        _case("adjoint_1024", "backward", "compensated", 1024, 1024, 4096, 0.3, 0.6),
        # A fitting step on the FP32 matrix cores.
        _case("step_1024_separable", "step", "separable", 1024, 1024, 4096, 0.3, 0.6),
        # The largest: one iteration of a 4K fit through autograd.
        _case("fit4k_autograd", "autograd", "compensated", 3840, 2160, 16384, 0.3, 0.6),
    ]


# Relative cost of one interaction by op and variant, so that a drawn case
# stays below the largest listed one.
_COST = {"plain": 2.0, "recurrence": 1.6, "compensated": 1.0, "separable": 0.5,
         "separable_f16x3": 0.25, "separable_f16": 0.2, "separable_bf16": 0.2}


def draw(rng):
    op = rng.choice(["forward", "forward", "noalloc", "step", "step", "backward", "autograd",
                     "f64"])
    variant = rng.choice(["compensated"] * 6 + ["separable_f16x3", "separable_f16x3",
                                                "separable_f16", "separable_bf16", "separable",
                                                "plain", "recurrence"])
    cost = (20.0 if op == "f64" else _COST[variant]) * (
        1.0 if op in ("forward", "noalloc", "f64") else 2.5)

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        nx, ny, n = log(128, 3840), log(96, 2160), log(64, 65536)
        if cost * nx * ny * n > 2.0e11:
            continue
        # the allocation-free call holds its scratch in 64 MiB
        if op == "noalloc" and cgh.workspace_bytes(n, nx, ny, variant) > cgh.NOALLOC_SCRATCH_BYTES:
            continue
        break
    zlo, zhi = rng.choice([(0.3, 0.6), (0.5, 1.0), (0.2, 1.5)])
    return _case(None, op, variant, nx, ny, n, zlo, zhi,
                 "mesh" if (zlo, zhi) == (0.2, 1.5) else "uniform")


# ------------------------------------------------------------------ inputs --

def _cloud(case, rng):
    """x, y, z, A in float64: uniform over the aperture, or on a height field
    of 17 x 10 random depths, bilinear in each cell."""
    nx, ny, n = case["nx"], case["ny"], case["n"]
    x, y = rng.uniform(0.0, nx, n), rng.uniform(0.0, ny, n)
    if case["cloud"] == "mesh":
        v = rng.uniform(case["zlo"], case["zhi"], (10, 17))
        u, w = x / nx * 16, y / ny * 9
        i, j = np.minimum(u.astype(int), 15), np.minimum(w.astype(int), 8)
        u, w = u - i, w - j
        z = ((1 - w) * ((1 - u) * v[j, i] + u * v[j, i + 1])
             + w * ((1 - u) * v[j + 1, i] + u * v[j + 1, i + 1]))
        return x, y, z, rng.uniform(0.0, 1.0, n)
    return x, y, rng.uniform(case["zlo"], case["zhi"], n), rng.uniform(0.5, 1.0, n)


def _tables(v, z, size):
    """cos and sin of P_j (h - v_j)^2 for h = 0 .. size - 1, float64 [n][size]."""
    prev = (PITCH * PITCH) / (2.0 * WAVELENGTH * z)
    h = torch.arange(size, dtype=torch.float64, device=v.device)
    rho = prev[:, None] * (h[None, :] - v[:, None]) ** 2
    t = 2.0 * math.pi * (rho - torch.round(rho))
    return torch.cos(t), torch.sin(t)


_CHUNK = 4096  # points at a time


def _hologram64(x, y, z, a, nx, ny):
    """Eq. (1) in float64: cos(X + Y) = cX cY - sX sY, one product per axis pair."""
    out = torch.zeros((ny, nx), dtype=torch.float64, device=x.device)
    for k in range(0, x.numel(), _CHUNK):
        s = slice(k, k + _CHUNK)
        cx, sx = _tables(x[s], z[s], nx)
        cy, sy = _tables(y[s], z[s], ny)
        out += torch.mm((a[s, None] * cy).t().contiguous(), cx)
        out -= torch.mm((a[s, None] * sy).t().contiguous(), sx)
    return out


def _gradients64(x, y, z, a, g):
    """dL/dx, dL/dy, dL/dz, dL/dA for G = dL/dI, float64."""
    ny, nx = g.shape
    hx = torch.arange(nx, dtype=torch.float64, device=x.device)
    hy = torch.arange(ny, dtype=torch.float64, device=x.device)
    parts = []
    for k in range(0, x.numel(), _CHUNK):
        s = slice(k, k + _CHUNK)
        cx, sx = _tables(x[s], z[s], nx)
        cy, sy = _tables(y[s], z[s], ny)
        u, v = torch.mm(cy, g), torch.mm(sy, g)          # sums over rows
        col = sx * u + cx * v                            # column sums of G sin
        gt = g.t().contiguous()
        row = cy * torch.mm(sx, gt) + sy * torch.mm(cx, gt)
        dx, dy = hx[None, :] - x[s, None], hy[None, :] - y[s, None]
        p = math.pi * PITCH * PITCH / (WAVELENGTH * z[s])
        sr = (col * dx * dx).sum(1) + (row * dy * dy).sum(1)
        parts.append((2 * a[s] * p * (col * dx).sum(1), 2 * a[s] * p * (row * dy).sum(1),
                      a[s] * p / z[s] * sr, (cx * u - sx * v).sum(1)))
    return tuple(torch.cat(c) for c in zip(*parts))


def _inputs(case, seed):
    """The float32 cloud, and T or G where the call takes one."""
    rng = np.random.default_rng(seed)
    dev = torch.device("cuda:0")
    hidden = _cloud(case, rng)

    def on_gpu(cols):
        return [torch.from_numpy(np.ascontiguousarray(c, dtype=np.float32)).to(dev)
                for c in cols]

    s = {}
    points = hidden
    if case["op"] in ("step", "backward", "autograd"):
        n = case["n"]
        points = (hidden[0] + rng.normal(0, 0.5, n), hidden[1] + rng.normal(0, 0.5, n),
                  hidden[2] + rng.normal(0, 1e-3, n), hidden[3] + rng.normal(0, 0.1, n))
        h = [c.double() for c in on_gpu(hidden)]
        s["target"] = _hologram64(*h, case["nx"], case["ny"]).float()
    s["points"] = on_gpu(points)
    if case["op"] == "backward":
        p64 = [c.double() for c in s["points"]]
        target = s.pop("target")
        s["grad"] = (_hologram64(*p64, case["nx"], case["ny"]) - target.double()).float()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["op"] == "noalloc":
        s["out"] = torch.empty((case["ny"], case["nx"]), dtype=torch.float32, device="cuda:0")
    if case["op"] == "autograd":
        x, y, z, a = s["points"]
        s["points"] = [x, y, z.requires_grad_(True), a.requires_grad_(True)]
    return s


def run(s):
    c = s["case"]
    x, y, z, a = s["points"]
    nx, ny, variant = c["nx"], c["ny"], c["variant"]
    op = c["op"]
    if op == "forward":
        return cgh.forward(x, y, z, a, nx, ny, PITCH, WAVELENGTH, variant)
    if op == "noalloc":
        return cgh.forward_noalloc(x, y, z, a, nx, ny, PITCH, WAVELENGTH, variant, out=s["out"])
    if op == "f64":
        return cgh.forward_f64(x, y, z, a, nx, ny, PITCH, WAVELENGTH)
    if op == "backward":
        return cgh.backward(x, y, z, a, s["grad"], nx, ny, PITCH, WAVELENGTH, variant)
    if op == "step":
        image, residual = cgh.forward_residual(x, y, z, a, s["target"], nx, ny, PITCH,
                                               WAVELENGTH, variant)
        grads = cgh.backward(x, y, z, a, residual, nx, ny, PITCH, WAVELENGTH, variant)
        return (image, residual) + tuple(grads)
    z.grad = a.grad = None
    image = cgh.CGHFunction.apply(x, y, z, a, nx, ny, PITCH, WAVELENGTH, variant)
    loss = 0.5 * torch.sum((image - s["target"]) ** 2)
    loss.backward()
    return image.detach(), loss.detach(), z.grad, a.grad


def exact(case, seed):
    s = _inputs(case, seed)
    p = [c.double() for c in s["points"]]
    nx, ny, op = case["nx"], case["ny"], case["op"]
    if op == "backward":
        return _gradients64(*p, s["grad"].double())
    image = _hologram64(*p, nx, ny)
    if op in ("forward", "noalloc", "f64"):
        return image
    residual = image - s["target"].double()
    grads = _gradients64(*p, residual)
    if op == "step":
        return (image, residual) + grads
    return image, 0.5 * (residual * residual).sum(), grads[2], grads[3]


def work(case):
    """Each input read once and each output written once; the sum as products
    of per-axis tables, two multiply-adds per point and pixel forward and four
    for the gradients (the least arithmetic of any form in the package)."""
    pixels, n, op = case["nx"] * case["ny"], case["n"], case["op"]
    grids, per_point, flops = {
        "forward": (1, 16, 4), "noalloc": (1, 16, 4), "f64": (2, 16, 4),
        "backward": (1, 32, 8), "step": (4, 48, 12), "autograd": (3, 40, 12)}[op]
    return {"bytes": 4.0 * grids * pixels + per_point * n, "flops": float(flops) * n * pixels}
