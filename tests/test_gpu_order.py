"""The order of addition of holograms of many points for their pixels.

Where the points' terms add up in phase, a residual I - T is a small difference
of large sums and shows their rounding, so the forwards keep one order of
addition there: the compensated and plain ones add the points one after the
other, the recurrence adds two halves of the points (padded to a multiple of 64)
so and then the two sums, and the separable ones add the points of each of
their plan's K splits so and then the splits.

At z = 1e30 every phase is below 1e-25 revolutions, every cosine 1 and every sine
lost against it, so a pixel is the sum of the amplitudes, which NumPy's running
FP32 sum gives to the bit in any stated order.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import device, say, to_dev
from paper_1002_0916_amd import binding as B
from paper_1002_0916_amd import workloads as W

pytestmark = pytest.mark.gpu


def cloud(n, nx, ny, seed):
    c = W.random_cloud(seed, n, nx, ny, alo=0.5, ahi=1.0)
    return W.Cloud(c.x, c.y, np.full(n, 1e30, dtype=np.float32), c.a)


def chain(a):
    """The FP32 sum of a, one after the other."""
    return np.add.accumulate(a.astype(np.float32), dtype=np.float32)[-1]


def check(c, nx, ny, variant, want):
    """I of all three entry points (where its scratch holds the problem, the
    allocation-free one too), and I - T, from the value of every pixel."""
    dev = device()
    say("order", (nx, ny, c.n), variant)
    x, y, z, a = to_dev(c, dev)
    T = torch.from_numpy(np.random.default_rng(7).standard_normal((ny, nx)).astype(np.float32))
    T = T.to(dev)
    I, G = B.forward_residual(x, y, z, a, T, nx, ny, variant=variant)
    J = B.forward(x, y, z, a, nx, ny, variant=variant)
    assert torch.equal(I, J) and torch.equal(G, I - T)
    if B.workspace_bytes(c.n, nx, ny, variant) <= B.NOALLOC_SCRATCH_BYTES:
        assert torch.equal(I, B.forward_noalloc(x, y, z, a, nx, ny, variant=variant))
    assert np.array_equal(I.cpu().numpy(), np.full((ny, nx), want, dtype=np.float32))


# The smallest number of points that keeps the order (24 n > pixels), remainders of
# the tiles and of 64 points, and many points on few pixels.
MANY = [(64, 48, 129), (130, 97, 526), (129, 95, 30001), (1, 1, 100), (365, 339, 10048)]


@pytest.mark.parametrize("shape", MANY)
def test_compensated_adds_the_points_in_order(shape):
    nx, ny, n = shape
    c = cloud(n, nx, ny, 2000 + n)
    check(c, nx, ny, "compensated", chain(c.a))


@pytest.mark.parametrize("shape", MANY)
def test_plain_adds_the_points_in_order(shape):
    nx, ny, n = shape
    c = cloud(n, nx, ny, 2100 + n)
    check(c, nx, ny, "plain", chain(c.a))


# The recurrence's lane shapes there: K = 4, 6 and 8 pixels, one and two rows.
@pytest.mark.parametrize("shape", MANY + [(133, 1130, 6300), (357, 628, 11209), (331, 1665, 23000),
                                          (441, 861, 18985), (437, 1109, 24231)])
def test_recurrence_adds_two_halves_in_order(shape):
    nx, ny, n = shape
    c = cloud(n, nx, ny, 2200 + n)
    half = -(-n // 64) * 32
    want = chain(c.a[:half])
    if n > half:
        want = np.float32(want + chain(c.a[half:]))
    check(c, nx, ny, "recurrence", want)


def splits(n, nx, ny):
    """The separable plans' K splits, restated: parts of whole stages of 16 points, at
    least 8 stages each, that minimise rounds of 512 tiles of 128 x 128 times the
    stages of a part, plus six stages of traffic a tile.  Points per part."""
    stages = -(-n // 64) * 4
    tiles = -(-nx // 128) * -(-ny // 128)
    best = (stages + 6 * tiles / 512 if tiles <= 512 else 0, stages)
    assert tiles <= 512
    for s in range(2, 513):
        per = -(-stages // s)
        if per < 8:
            break
        if -(-stages // per) == s:
            t = -(-tiles * s // 512) * per + 6 * s * tiles / 512
            best = min(best, (t, per), key=lambda v: v[0])
    return 16 * best[1]


# One point of 16 has an amplitude, of 8 bits between 2^-14 and 1 (exact in every
# format), so that a matrix instruction adds one number to its sum.
@pytest.mark.parametrize("variant", ["separable", "separable_f16x3", "separable_f16",
                                     "separable_bf16"])
@pytest.mark.parametrize("shape", [(64, 48, 1025), (130, 97, 4204), (129, 95, 60001),
                                   (1, 1, 5000), (257, 300, 25701)])
def test_separable_adds_its_splits_in_order(variant, shape):
    nx, ny, n = shape
    assert 3 * n > nx * ny
    c = cloud(n, nx, ny, 2300 + n)
    rng = np.random.default_rng(2301 + n)
    a = np.zeros(n, dtype=np.float32)
    at = np.arange(0, n - 15, 16) + rng.integers(0, 16, n // 16)
    a[at] = np.ldexp(rng.integers(128, 256, at.size), rng.integers(-21, -7, at.size))
    per = splits(n, nx, ny)
    want = chain(np.array([chain(a[k:k + per]) for k in range(0, n, per)]))
    check(W.Cloud(c.x, c.y, c.z, a), nx, ny, variant, want)
