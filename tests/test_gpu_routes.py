"""The forward contraction's routes against the FP64 hologram, by the 2-norm of the
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

from gpu_helpers import U_BF16, U_F16, device, say, to_dev
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
