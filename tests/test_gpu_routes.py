"""The contractions' routes against FP64 ones, the forward by the 2-norm of the
error over the whole grid: slices and chunks of points, and few points on very many
pixels.

The error is relative to the hologram.  A term of the f16x3 format is off by
independent roundings: two phases (each 2 pi 2^-24 (1 + 1.5 Prev |m|) at most, a
third of it in the mean square), four native cosines and sines (2.5e-7 at most) and
the planes (2^-23): together below 4e-7 in the mean square at the sizes here.  An
addition to a sum S is off by up to 2^-25 |S|; in a chain of 3 n / 16 additions (half
the points, three products of 8 at a time) that grows to 1.8e-8 sqrt(3 n / 16) of a
sum in phase, and less otherwise.  The single planes' operands are off by up to u =
2^-11 or 2^-8 each, a third of it in the mean square, and a term has two.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import U_BF16, U_F16, device, rel_l2, say, to_dev
from paper_1002_0916_amd import binding as B
from paper_1002_0916_amd import workloads as W

pytestmark = pytest.mark.gpu


def bar(variant, n):
    planes = {"separable_f16": U_F16, "separable_bf16": U_BF16}.get(variant, 0.0)
    return planes + 4e-7 + 1.8e-8 * (3 * n / 16) ** 0.5


def error(c, nx, ny, variant):
    """2-norm of I - I64 over that of I64, and I."""
    p = to_dev(c, device())
    I = B.forward(*p, nx, ny, variant=variant)
    ref = B.forward_f64(*p, nx, ny)
    return ((I.double() - ref).norm() / ref.norm()).item(), I


def check(variant, shape, seed):
    nx, ny, n = shape
    say("forward route", shape, variant)
    c = W.random_cloud(seed + n, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0)
    e, _ = error(c, nx, ny, variant)
    say("  rel-L2 = %.2e, bar %.2e" % (e, bar(variant, n)))
    assert e <= bar(variant, n)


# Few points on many pixels, where the tiles' stores weigh: the largest tile, and its
# remainders (beyond 2^23 pixels, 5 2^20 for the single planes, any in FP32).
@pytest.mark.parametrize("variant,shape", [
    ("separable_f16", (6029, 4883, 9)), ("separable_bf16", (3839, 2159, 200)),
    ("separable_f16x3", (4100, 2113, 65)), ("compensated", (4100, 2113, 9)),
    ("separable", (3840, 2160, 64)), ("separable", (701, 333, 30))])
def test_few_points_on_many_pixels(variant, shape):
    check(variant, shape, 2400)


# Points in slices and in chunks whose tables fit, the last one shorter
# (tests/test_plans.py states the routes).
SLICES = [("compensated", (700, 500, 9001)), ("separable_f16x3", (400, 300, 4901)),
          ("separable", (256, 200, 12001)), ("separable_f16", (640, 480, 90001)),
          ("separable_bf16", (1382, 471, 36661)), ("compensated", (1920, 1080, 65537)),
          ("compensated", (1100, 1500, 65001))]


@pytest.mark.parametrize("variant,shape", SLICES)
def test_slices_and_chunks(variant, shape):
    check(variant, shape, 2500)


@pytest.mark.parametrize("variant,shape", SLICES)
def test_the_last_points_count(variant, shape):
    """Only the last 1, 2, ... 64 points have an amplitude: the hologram is that of
    those points alone, up to two routes' rounding."""
    nx, ny, n = shape
    say("last points", shape, variant)
    c = W.random_cloud(2600 + n, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0)
    for last in (1, 2, 17, 64):
        a = c.a.copy()
        a[:n - last] = 0.0
        I = B.forward(*to_dev(W.Cloud(c.x, c.y, c.z, a), device()), nx, ny, variant=variant)
        alone = W.Cloud(*(v[n - last:] for v in c.astuple()))
        J = B.forward(*to_dev(alone, device()), nx, ny, variant=variant)
        e = ((I.double() - J.double()).norm() / J.double().norm()).item()
        say("  %d: rel-L2 = %.2e" % (last, e))
        assert e <= 2 * bar(variant, last)


@pytest.mark.parametrize("variant", ["compensated", "separable_f16x3"])
@pytest.mark.parametrize("shape", [(1024, 1024, 1000), (333, 197, 700), (256, 256, 64),
                                   (700, 500, 9001)])
def test_low_planes_count(variant, shape):
    """hi + lo operands are some 2^11 times as exact as hi alone: a lost product of a low
    plane would leave an error of f16's size."""
    nx, ny, n = shape
    say("low planes", shape, variant)
    c = W.random_cloud(2700 + n, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0)
    e, _ = error(c, nx, ny, variant)
    one, _ = error(c, nx, ny, "separable_f16")
    say("  rel-L2 = %.2e, f16 %.2e" % (e, one))
    assert e <= one / 200


@pytest.mark.parametrize("variant", ["compensated", "separable_f16x3"])
@pytest.mark.parametrize("shape", [(1024, 1024, 1000), (1920, 1080, 300), (700, 500, 9001)])
def test_scale_of_the_hologram(variant, shape):
    """The native cosine and sine are 3.3e-8 too small in the mean, a product of two of
    them 6.6e-8, which one operand's factor 1 + 2^-24 takes back: the hologram's scale
    (its regression on the FP64 one) is off by less than half of what it was."""
    nx, ny, n = shape
    c = W.random_cloud(2800 + n, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0)
    p = to_dev(c, device())
    I = B.forward(*p, nx, ny, variant=variant).double()
    ref = B.forward_f64(*p, nx, ny)
    off = ((I * ref).sum() / (ref * ref).sum() - 1).item()
    say("scale", shape, variant, "%.2e" % off)
    assert abs(off) < 3.3e-8


# The adjoint, tiled and one tile a workgroup; G everywhere, and in the last row and
# column alone (the remainders of every tile, stage and step).
@pytest.mark.parametrize("variant", ["compensated", "separable_f16x3", "separable"])
@pytest.mark.parametrize("shape", [(1501, 1037, 1300), (333, 197, 700), (129, 65, 33)])
@pytest.mark.parametrize("edge", [False, True])
def test_adjoint_counts_low_planes_and_edges(oracle_mod, variant, shape, edge):
    """The gradients' relative error is that of the forward's terms (a gradient and its
    error sum the same terms), and some 2^11 times below f16's."""
    nx, ny, n = shape
    dev = device()
    say("adjoint", shape, variant, "edge" if edge else "")
    c = W.random_cloud(2900 + n, n, nx, ny, zlo=0.3, zhi=1.0, alo=0.5, ahi=1.0)
    G = np.random.default_rng(n).standard_normal((ny, nx)).astype(np.float32)
    if edge:
        G[:-1, :-1] = 0.0
    idx = np.arange(0, n, max(1, n // 100))
    ref = oracle_mod.adjoint(*c.astuple(), nx, ny, G, idx=idx, threads=0)
    g = torch.from_numpy(G).to(dev)

    def errors(v):
        grads = B.backward(*to_dev(c, dev), g, nx, ny, variant=v)
        return [rel_l2(t.cpu().numpy()[idx], r) for t, r in zip(grads, ref)]

    e, one = errors(variant), errors("separable_f16")
    say("  rel-L2", " ".join("%.1e" % v for v in e), "f16", " ".join("%.1e" % v for v in one))
    assert max(e) <= bar(variant, max(nx, ny)) and max(e) <= min(one) / 100
