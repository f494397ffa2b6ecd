"""Infinities and NaN in the inputs of the contraction kernels: what one element
gives stays that element's, at the edges of the hologram and of the tiles too."""
import numpy as np
import pytest
import torch

from gpu_helpers import device, say, to_dev
from paper_1002_0916_amd import binding as B
from paper_1002_0916_amd import workloads as W

pytestmark = pytest.mark.gpu

SEPARABLE = ["separable", "separable_f16", "separable_bf16"]


def axis_cos_sin(c, axis, at):
    """cos and sin of each point's phase on one axis at pixel `at`, float64."""
    v = (c.x if axis == "x" else c.y).astype(np.float64)
    rho = W.PITCH ** 2 / (2 * W.WAVELENGTH * c.z.astype(np.float64)) * (at - v) ** 2
    return np.cos(2 * np.pi * rho), np.sin(2 * np.pi * rho)


# Tiled (1200x900) and one tile a workgroup (150x110); the last pixel, the last row
# and column, and one inside.
@pytest.mark.parametrize("variant", SEPARABLE)
@pytest.mark.parametrize("shape", [(1201, 903, 1000), (150, 110, 40)])
@pytest.mark.parametrize("where", ["corner", "row", "column", "inside"])
def test_adjoint_infinite_gradient_in_separable_form(variant, shape, where):
    """dL/dA_j = sum_x (cX U - sX V), U = sum_y G cY, V = sum_y G sY: an infinite G
    makes both terms of its column infinite, and the difference the first one's
    infinity or, where they have one sign, NaN."""
    nx, ny, n = shape
    dev = device()
    say("infinite G", shape, variant, where)
    c = W.random_cloud(1701, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0)
    px = nx - 1 if where in ("corner", "column") else nx // 3
    py = ny - 1 if where in ("corner", "row") else ny // 3
    g = torch.from_numpy(np.random.default_rng(5).standard_normal((ny, nx)).astype(np.float32))
    g = g.to(dev)
    g[py, px] = float("inf")
    ga = B.backward(*to_dev(c, dev), g, nx, ny, variant=variant)[3].cpu().numpy()
    (cx, sx), (cy, sy) = axis_cos_sin(c, "x", px), axis_cos_sin(c, "y", py)
    clear = np.min(np.abs([cx, sx, cy, sy]), axis=0) > 1e-2
    want = np.where(cx * cy * sx * sy > 0, np.nan, np.where(cx * cy > 0, np.inf, -np.inf))
    assert clear.sum() > n // 2 and np.isinf(want[clear]).any()
    assert np.array_equal(ga[clear], want[clear].astype(np.float32), equal_nan=True)


# One launch from the points, tables with max |A| found by each workgroup (up to 8192
# points) and by a launch of its own, and sums in the order of the points.
@pytest.mark.parametrize("variant", SEPARABLE)
@pytest.mark.parametrize("shape", [(150, 110, 40), (400, 330, 5000), (400, 330, 9000),
                                   (70, 50, 9000)])
def test_forward_infinite_amplitude_in_separable_form(variant, shape):
    """A (cY cX - sY sX) with an infinite A: the first product's infinity or, where
    both products have one sign, NaN."""
    nx, ny, n = shape
    dev = device()
    say("infinite A", shape, variant)
    c = W.random_cloud(1703, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0)
    x, y, z, a = to_dev(c, dev)
    a[n - 2] = float("inf")
    I = B.forward(x, y, z, a, nx, ny, variant=variant).cpu().numpy()
    cs = {}
    for axis, v, size in (("x", c.x, nx), ("y", c.y, ny)):
        rho = (W.PITCH ** 2 / (2 * W.WAVELENGTH * float(c.z[n - 2]))
               * (np.arange(size) - float(v[n - 2])) ** 2)
        cs[axis] = np.cos(2 * np.pi * rho), np.sin(2 * np.pi * rho)
    cc, ss = (np.outer(cs["y"][k], cs["x"][k]) for k in (0, 1))
    clear = np.outer(np.min(np.abs(cs["y"]), axis=0) > 1e-2, np.min(np.abs(cs["x"]), axis=0) > 1e-2)
    want = np.where(cc * ss > 0, np.nan, np.where(cc > 0, np.inf, -np.inf)).astype(np.float32)
    assert clear.sum() > nx * ny // 4
    assert np.array_equal(I[clear], want[clear], equal_nan=True)


def best_ms(f):
    f()
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.parametrize("variant", ["compensated", "separable_f16x3"])
def test_nan_costs_what_finite_values_do(variant):
    """A NaN amplitude or gradient makes every result NaN without a sum term by term
    (which takes 30 to 40 times as long here)."""
    dev = device()
    nx, ny, n = 1920, 1080, 8192
    x, y, z, a = to_dev(W.random_cloud(1702, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0), dev)
    g = torch.from_numpy(np.random.default_rng(6).standard_normal((ny, nx)).astype(np.float32))
    g = g.to(dev)
    out = torch.empty((ny, nx), device=dev)
    forward = lambda: B.forward(x, y, z, a, nx, ny, variant=variant, out=out)
    backward = lambda: B.backward(x, y, z, a, g, nx, ny, variant=variant)
    finite = best_ms(forward), best_ms(backward)
    g[3, 5] = float("nan")
    grads = backward()
    assert all(torch.isnan(t).all() for t in grads)
    nan_g = best_ms(backward)
    a[7] = float("nan")
    assert torch.isnan(forward()).all()
    say("NaN", variant, "forward, backward ms:", finite, (best_ms(forward), nan_g))
    assert best_ms(forward) < 5 * finite[0] and nan_g < 5 * finite[1]
