"""The contraction kernels (operands formed in the kernel, matrix cores) and the
plain forward: every tile shape and point split of the forward and the adjoint's
tiles, slices and column groups, at their edges, and the inputs the formats
treat specially.

Tolerance of the f16x3 format against the FP64 oracle, as a fraction of
sum |A|.  A table value is off by 2 pi times its phase error (about
2^-24 (1 + 1.5 Prev |m|) revolutions, Prev = p^2 / (2 lambda z), |m| the largest
offset), the transcendental's own error (below 2.5e-7) and the planes'
rounding (2^-23); a term is two products of two such values, so four of these.
Adding in FP32 costs at most 2^-24 per addition in a wave's chain (three per 8
points of its share).
"""
import numpy as np
import pytest
import torch

from gpu_helpers import (TOL_ADJ, TOL_FWD, device, max_err_frac, rel_l2, say, to_dev,
                         upstream_gradient)
from paper_1002_0916_amd import binding as B
from paper_1002_0916_amd import workloads as W

pytestmark = pytest.mark.gpu

ZLO = 0.3


def f16x3_bar(nx, ny, n, margin):
    prev = W.PITCH ** 2 / (2 * W.WAVELENGTH * ZLO)
    phase = 2 * np.pi * 2.0 ** -24 * (1 + 1.5 * prev * (max(nx, ny) + margin))
    return 4 * (phase + 2.5e-7 + 2.0 ** -23) + 2.0 ** -24 * 3 * (n / 8 + 8)


# (nx, ny, n): one step and its neighbours; remainders of 32 and 64 in every
# size; each tile shape (32x32, 32x64, 64x64, 64x128 and 128x128 pixels); the
# points in several slices (128x96 and 40x20).
FORWARD = [(32, 32, 9), (33, 31, 64), (65, 129, 65), (333, 197, 700), (600, 500, 1500),
           (1024, 1024, 1000), (1920, 1080, 1000), (3840, 2160, 100), (128, 96, 5000),
           (40, 20, 3001)]


@pytest.mark.parametrize("variant", ["compensated", "separable", "separable_f16x3",
                                     "separable_f16", "separable_bf16"])
@pytest.mark.parametrize("shape", FORWARD)
def test_forward_shapes(oracle_mod, variant, shape):
    nx, ny, n = shape
    dev = device()
    say("contraction forward", shape, variant)
    c = W.random_cloud(1000 + n, n, nx, ny, zlo=ZLO, zhi=1.0, alo=-1.0, ahi=1.0, margin=20)
    x, y, z, a = to_dev(c, dev)
    rng = np.random.default_rng(n)
    T = torch.from_numpy(rng.standard_normal((ny, nx)).astype(np.float32)).to(dev)
    I, G = B.forward_residual(x, y, z, a, T, nx, ny, variant=variant)
    J = B.forward(x, y, z, a, nx, ny, variant=variant)
    torch.cuda.synchronize()
    assert torch.equal(I, J) and torch.equal(G, I - T)
    px, py = W.sample_pixels(1001, nx, ny, 3000)
    ref = oracle_mod.forward_at(*c.astuple(), nx, ny, px, py, threads=0)
    err = max_err_frac(I.cpu().numpy()[py, px], ref, c)
    bar = (f16x3_bar(nx, ny, n, 20) if variant in ("compensated", "separable_f16x3")
           else TOL_FWD[variant])
    say("  max|dI|/sum|A| = %.3e, bar %.3e" % (err, bar))
    assert err <= bar


# One launch without tables: one point and the records' rounds of 512 with their
# neighbours, tiles of 32 pixels and remainders (compensated calls of up to 8
# points take the direct sum).
@pytest.mark.parametrize("variant", ["compensated", "separable", "separable_f16x3",
                                     "separable_f16", "separable_bf16"])
@pytest.mark.parametrize("shape", [(33, 31, 1), (32, 32, 9), (65, 97, 511), (100, 40, 513),
                                   (256, 256, 1024), (256, 256, 1025), (1920, 1080, 16)])
def test_forward_few_points(oracle_mod, variant, shape):
    test_forward_shapes(oracle_mod, variant, shape)


# Tables in chunks of points, the last one shorter, without and with slices in a
# chunk: the compensated variant's where the column table of all points has no room,
# the single planes' where both tables exceed 256 MiB.
@pytest.mark.parametrize("variant,shape", [("compensated", (1024, 700, 65601)),
                                           ("compensated", (1273, 331, 91466)),
                                           ("separable_f16", (1920, 1080, 24001)),
                                           ("separable_bf16", (1382, 471, 36660))])
def test_forward_chunks(oracle_mod, variant, shape):
    nx, ny, n = shape
    assert (nx if variant == "compensated" else nx + ny) * n * 4 > 256 << 20
    test_forward_shapes(oracle_mod, variant, shape)


@pytest.mark.parametrize("scale", [1e-30, 1e30])
def test_forward_amplitudes_of_any_scale(oracle_mod, scale):
    """One amplitude 2^20 times the others, at both ends of the FP32 range."""
    dev = device()
    nx, ny, n = 150, 110, 200
    c = W.random_cloud(1101, n, nx, ny, zlo=ZLO, zhi=1.0, alo=-1.0, ahi=1.0, margin=15)
    a = c.a.astype(np.float64) * scale * 2.0 ** -20
    a[7] = scale
    c = W.Cloud(c.x, c.y, c.z, a.astype(np.float32))
    I = B.forward(*to_dev(c, dev), nx, ny, variant="compensated").cpu().numpy()
    ref = oracle_mod.forward(*c.astuple(), nx, ny, threads=0)
    err = max_err_frac(I, ref, c)
    say("amplitude scale", scale, "max|dI|/sum|A| =", err)
    assert np.all(np.isfinite(I)) and err <= f16x3_bar(nx, ny, n, 15)


@pytest.mark.parametrize("shape", [(70, 50, 20), (70, 50, 600), (128, 96, 2000)])
def test_forward_non_finite_amplitudes(shape):
    """An infinite amplitude gives the infinities of its term's cosine, a NaN
    gives NaN everywhere, as the sum term by term does."""
    dev = device()
    nx, ny, n = shape
    c = W.random_cloud(1102, n, nx, ny, zlo=ZLO, zhi=1.0, alo=0.5, ahi=1.0)
    x, y, z, a = to_dev(c, dev)
    a[3] = float("inf")
    I = B.forward(x, y, z, a, nx, ny, variant="compensated").cpu().numpy()
    h, v = np.meshgrid(np.arange(nx), np.arange(ny))
    P = np.pi * W.PITCH ** 2 / (W.WAVELENGTH * float(c.z[3]))
    cos = np.cos(P * ((h - float(c.x[3])) ** 2 + (v - float(c.y[3])) ** 2))
    clear = np.abs(cos) > 1e-3
    assert np.array_equal(I[clear], np.where(cos > 0, np.inf, -np.inf)[clear])
    a[3] = float("nan")
    assert torch.isnan(B.forward(x, y, z, a, nx, ny, variant="compensated")).all()


# (nx, ny, n): tiles of 128 coordinates, stages of 32 and steps of 16 with their
# remainders on both axes, blocks of 128 points with theirs; several tiles per
# workgroup (640x100) and a single short one.
ADJOINT = [(32, 32, 9), (33, 32, 64), (65, 129, 65), (129, 127, 200), (333, 197, 700),
           (640, 100, 3000), (40, 1500, 129), (1501, 37, 130)]
# The direct kernel: tiles of 32, steps of 16 and rounds of eight steps with their
# remainders; several tiles a workgroup (2000x33 with few planes).
ADJOINT += [(32, 33, 1), (16, 129, 33), (127, 128, 32), (250, 40, 64), (2000, 33, 9)]


@pytest.mark.parametrize("variant", ["compensated", "separable", "separable_f16x3",
                                     "separable_f16", "separable_bf16"])
@pytest.mark.parametrize("shape", ADJOINT)
def test_adjoint_shapes(oracle_mod, variant, shape):
    """The f16x3 bar is the forward's, with the chain of additions over the
    longer side (three per 16 coordinates); a sum of many terms of either sign
    and its error grow alike, so the bar holds for the relative L2 error."""
    nx, ny, n = shape
    dev = device()
    say("contraction adjoint", shape, variant)
    c = W.random_cloud(1200 + n, n, nx, ny, zlo=ZLO, zhi=1.0, alo=0.5, ahi=1.0, margin=20)
    G = upstream_gradient(oracle_mod, nx, ny, 1201)
    # G at an address that is a multiple of 4 bytes only
    flat = torch.empty(nx * ny + 1, device=dev)
    g = flat[1:].view(ny, nx)
    g.copy_(torch.from_numpy(G))
    grads = B.backward(*to_dev(c, dev), g, nx, ny, variant=variant)
    again = B.backward(*to_dev(c, dev), g, nx, ny, variant=variant)
    idx = np.arange(0, n, max(1, n // 200))
    ref = oracle_mod.adjoint(*c.astuple(), nx, ny, G, idx=idx, threads=0)
    bar = (f16x3_bar(nx, ny, max(nx, ny) / 2, 20)
           if variant in ("compensated", "separable_f16x3") else TOL_ADJ[variant])
    for name, t, u, r in zip("xyza", grads, again, ref):
        assert torch.equal(t, u)
        e = rel_l2(t.cpu().numpy()[idx], r)
        say("  d%s rel-L2 = %.3e, bar %.3e" % (name, e, bar))
        assert e <= bar


@pytest.mark.parametrize("shape", [(70, 150, 200), (700, 450, 400)])
def test_adjoint_non_finite_gradient(shape):
    """An infinite G gives each point the infinity of its term, a NaN gives NaN."""
    dev = device()
    nx, ny, n = shape
    c = W.random_cloud(1301, n, nx, ny, zlo=ZLO, zhi=1.0, alo=0.5, ahi=1.0)
    x, y, z, a = to_dev(c, dev)
    g = torch.from_numpy(np.random.default_rng(3).standard_normal((ny, nx)).astype(np.float32))
    g = g.to(dev)
    px, py = 61, 140
    g[py, px] = float("inf")
    ga = B.backward(x, y, z, a, g, nx, ny, variant="compensated")[3].cpu().numpy()
    P = np.pi * W.PITCH ** 2 / (W.WAVELENGTH * c.z.astype(np.float64))
    cos = np.cos(P * ((px - c.x.astype(np.float64)) ** 2 + (py - c.y.astype(np.float64)) ** 2))
    clear = np.abs(cos) > 1e-3
    assert np.array_equal(ga[clear], np.where(cos > 0, np.inf, -np.inf)[clear])
    g[py, px] = float("nan")
    for t in B.backward(x, y, z, a, g, nx, ny, variant="compensated"):
        assert torch.isnan(t).all()


@pytest.mark.parametrize("shape", [(150, 110, 100), (700, 450, 400)])
@pytest.mark.parametrize("scale", [1e-30, 1e30])
def test_adjoint_gradient_of_any_scale(oracle_mod, shape, scale):
    """One pixel 2^20 times the others, at both ends of the FP32 range."""
    dev = device()
    nx, ny, n = shape
    c = W.random_cloud(1302, n, nx, ny, zlo=ZLO, zhi=1.0, alo=0.5, ahi=1.0)
    G = np.random.default_rng(5).standard_normal((ny, nx)) * scale * 2.0 ** -20
    G[40, 77] = scale
    G = G.astype(np.float32)
    ga = B.backward(*to_dev(c, dev), torch.from_numpy(G).to(dev), nx, ny,
                    variant="compensated")[3].cpu().numpy()
    ref = oracle_mod.adjoint(*c.astuple(), nx, ny, G, threads=0)[3]
    e = rel_l2(ga.astype(np.float64) / scale, ref / scale)
    say("gradient scale", scale, "rel-L2 =", e)
    assert np.all(np.isfinite(ga)) and e <= f16x3_bar(nx, ny, nx / 2, 0)


# Tiles of 64 pixels and their remainders; the points in slices (128x96) and in
# chunks whose tables fit (3840x2160, two chunks).
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 65, 64), (333, 197, 700), (128, 96, 3001),
                                   (3840, 2160, 1400)])
def test_f64_shapes(oracle_mod, shape):
    """A phase is at most about 2600 revolutions here, so its FP64 rounding is
    below 2 pi 2600 2^-52 = 3.6e-12 of a term; the sum adds less."""
    nx, ny, n = shape
    dev = device()
    say("f64", shape)
    c = W.random_cloud(1400 + n, n, nx, ny, zlo=ZLO, zhi=1.0, alo=-1.0, ahi=1.0)
    I = B.forward_f64(*to_dev(c, dev), nx, ny)
    assert torch.equal(I, B.forward_f64(*to_dev(c, dev), nx, ny))
    px, py = W.sample_pixels(1401, nx, ny, 2000)
    ref = oracle_mod.forward_at(*c.astuple(), nx, ny, px, py, threads=0)
    err = max_err_frac(I.cpu().numpy()[py, px], ref, c)
    say("  max|dI|/sum|A| = %.3e" % err)
    assert err <= 1e-11


def test_f64_non_finite_amplitudes():
    dev = device()
    nx, ny = 70, 50
    c = W.random_cloud(1402, 20, nx, ny, zlo=ZLO, zhi=1.0, alo=0.5, ahi=1.0)
    x, y, z, a = to_dev(c, dev)
    a[3] = float("-inf")
    I = B.forward_f64(x, y, z, a, nx, ny).cpu().numpy()
    h, v = np.meshgrid(np.arange(nx), np.arange(ny))
    P = np.pi * W.PITCH ** 2 / (W.WAVELENGTH * float(c.z[3]))
    cos = np.cos(P * ((h - float(c.x[3])) ** 2 + (v - float(c.y[3])) ** 2))
    clear = np.abs(cos) > 1e-6
    assert np.array_equal(I[clear], np.where(cos > 0, -np.inf, np.inf)[clear])
    a[3] = float("nan")
    assert torch.isnan(B.forward_f64(x, y, z, a, nx, ny)).all()


# The recurrence forward: each K (4, 6 and 8 pixels) with each of 1, 2 and 4 rows
# per lane, tiles of 64 points and parts of 8 with their remainders.
@pytest.mark.parametrize("shape", [(1, 1, 1), (70, 50, 9), (333, 197, 65), (3840, 2160, 7),
                                   (3520, 13, 63), (640, 480, 129), (1640, 1333, 33),
                                   (2368, 16, 64), (2480, 184, 100), (1920, 1024, 70)])
def test_recurrence_forward_shapes(oracle_mod, shape):
    """The plain phase's five roundings at the first pixel of a lane, and those of
    seven steps of Gamma and delta (each below 64 revolutions)."""
    nx, ny, n = shape
    dev = device()
    say("recurrence forward", shape)
    c = W.random_cloud(1600 + n, n, nx, ny, zlo=ZLO, zhi=1.0, alo=-1.0, ahi=1.0, margin=20)
    x, y, z, a = to_dev(c, dev)
    T = torch.from_numpy(np.random.default_rng(n).standard_normal((ny, nx)).astype(np.float32))
    T = T.to(dev)
    I, G = B.forward_residual(x, y, z, a, T, nx, ny, variant="recurrence")
    J = B.forward(x, y, z, a, nx, ny, variant="recurrence")
    assert torch.equal(I, J) and torch.equal(G, I - T)
    px, py = W.sample_pixels(1601, nx, ny, 3000)
    ref = oracle_mod.forward_at(*c.astuple(), nx, ny, px, py, threads=0)
    err = max_err_frac(I.cpu().numpy()[py, px], ref, c)
    prev = W.PITCH ** 2 / (2 * W.WAVELENGTH * ZLO)
    revs = 5 * prev * ((nx + 20) ** 2 + (ny + 20) ** 2)        # Gamma_0
    revs += 7 * 3 * prev * 2 * (nx + 20)                       # delta_0, seven times
    revs += 2 * 7 * 64                                         # the steps' additions
    bar = 2 * np.pi * 2.0 ** -24 * revs + 2.5e-7 + 2.0 ** -24 * (n + 8)
    say("  max|dI|/sum|A| = %.3e, bar %.3e" % (err, bar))
    assert err <= bar


# The plain forward: rows per lane, groups that split the points and tiles of 64
# points with their remainders (each of the rule's three forms); phases within and
# beyond the cosine's exact range of 256 revolutions (3840 columns reach 2500).
@pytest.mark.parametrize("shape", [(1, 1, 1), (63, 7, 63), (65, 9, 65), (640, 490, 300),
                                   (1024, 603, 129), (3841, 1100, 70)])
def test_plain_forward_shapes(oracle_mod, shape):
    """Five roundings of 2^-24 of the phase (dx or dy twice in its square, the
    sum, Prev, the product) and the cosine's 2.5e-7."""
    nx, ny, n = shape
    dev = device()
    say("plain forward", shape)
    c = W.random_cloud(1500 + n, n, nx, ny, zlo=ZLO, zhi=1.0, alo=-1.0, ahi=1.0, margin=20)
    x, y, z, a = to_dev(c, dev)
    T = torch.from_numpy(np.random.default_rng(n).standard_normal((ny, nx)).astype(np.float32))
    T = T.to(dev)
    I, G = B.forward_residual(x, y, z, a, T, nx, ny, variant="plain")
    J = B.forward(x, y, z, a, nx, ny, variant="plain")
    assert torch.equal(I, J) and torch.equal(G, I - T)
    px, py = W.sample_pixels(1501, nx, ny, 3000)
    ref = oracle_mod.forward_at(*c.astuple(), nx, ny, px, py, threads=0)
    err = max_err_frac(I.cpu().numpy()[py, px], ref, c)
    revs = W.PITCH ** 2 / (2 * W.WAVELENGTH * ZLO) * ((nx + 20) ** 2 + (ny + 20) ** 2)
    bar = 2 * np.pi * 5 * 2.0 ** -24 * revs + 2.5e-7 + 2.0 ** -24 * (n + 8)
    say("  max|dI|/sum|A| = %.3e, bar %.3e" % (err, bar))
    assert err <= bar
