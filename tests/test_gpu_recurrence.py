"""The recurrence forward, every instance of its kernel: K = 4, 6 and 8 pixels and 1, 2
or 4 rows per lane, eight parts of the points or (many points on few pixels) two."""
import numpy as np
import pytest

from gpu_helpers import device, max_err_frac, say, to_dev
from paper_1002_0916_amd import binding as B
from paper_1002_0916_amd import workloads as W

pytestmark = pytest.mark.gpu


def instance(nx, ny, n):
    """The launcher's rule, restated: (K, rows, parts)."""
    def up(a, b):
        return -(-a // b)

    best = None
    for k, r in ((8, 4), (8, 2), (8, 1), (6, 4), (6, 2), (6, 1), (4, 4), (4, 2), (4, 1)):
        wgs = up(nx, 64 * k) * up(ny, 4 * r)
        t = up(wgs, 256) * k * r * (4 + 1 / r + (4 * r + 7) / (k * r))
        if best is None or t < best[0]:
            best = (t, k)
    k = best[1]
    cols = up(nx, 64 * k)
    if 24 * n > nx * ny:
        one, two = up(cols * up(ny, 4), 256), up(cols * up(ny, 8), 256)
        return k, 1 if 10 * one < 17 * two else 2, 2
    waves = cols * up(ny, 4)
    if k == 4 and waves <= 80:
        return k, 1, 8
    return k, 2 if waves <= 430 else 4, 8


SHAPES = [(160, 245, 20), (505, 403, 65), (1101, 1153, 33), (357, 628, 100), (968, 1803, 73),
          (441, 861, 33), (3839, 2161, 10), (64, 48, 129), (137, 1131, 6500), (357, 629, 9400),
          (331, 1667, 23001), (441, 863, 15901), (437, 1109, 20201)]


def test_every_instance_is_tested():
    assert {instance(*s) for s in SHAPES} == (
        {(4, 1, 8)} | {(k, r, 8) for k in (4, 6, 8) for r in (2, 4)}
        | {(k, r, 2) for k in (4, 6, 8) for r in (1, 2)})


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%d-%d" % s)
def test_recurrence_instances(oracle_mod, shape):
    """The plain phase's five roundings at a lane's first pixel, those of seven steps of
    Gamma and delta (each below 64 revolutions), and an FP32 sum (test_gpu_contract.py)."""
    nx, ny, n = shape
    say("recurrence", shape, "instance", instance(*shape))
    c = W.random_cloud(3000 + n, n, nx, ny, zlo=0.3, zhi=1.0, alo=-1.0, ahi=1.0, margin=20)
    I = B.forward(*to_dev(c, device()), nx, ny, variant="recurrence").cpu().numpy()
    px, py = W.sample_pixels(3001, nx, ny, 400)
    ref = oracle_mod.forward_at(*c.astuple(), nx, ny, px, py, threads=0)
    err = max_err_frac(I[py, px], ref, c)
    prev = W.PITCH ** 2 / (2 * W.WAVELENGTH * 0.3)
    revs = 5 * prev * ((nx + 20) ** 2 + (ny + 20) ** 2) + 7 * 3 * prev * 2 * (nx + 20) + 2 * 7 * 64
    bar = 2 * np.pi * 2.0 ** -24 * revs + 2.5e-7 + 2.0 ** -24 * (n + 8)
    say("  max|dI|/sum|A| = %.3e, bar %.3e" % (err, bar))
    assert err <= bar
