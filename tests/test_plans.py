"""The library's plans, on the host (no GPU needed, no kernel launched): every launch
within HIP's limits, no empty slice, and the regions that a route uses apart from each
other inside the workspace; and the routes that the GPU tests of them are meant to
take.  tests/plans/check.hip calls the planning functions of libcgh.so."""
import math
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_1002_0916_amd")
HBM = 288 << 30
FORWARD, FORWARD_F64, BACKWARD = 0, 1, 2
COMPENSATED, SEPARABLE, F16X3, F16, BF16 = 1, 2, 3, 4, 5


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    from paper_1002_0916_amd import build

    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path_factory.mktemp("plans") / "check")
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-std=c++17",
                    "-O1", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "plans", "check.hip"), "-L", PKG, "-lcgh",
                    "-Wl,-rpath," + PKG, "-o", exe], check=True, capture_output=True)

    def run(calls):
        """One line per (variant, op, nx, ny, n, column table)."""
        text = "".join("%d %d %d %d %d %d\n" % tuple(map(int, c)) for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        lines = out.stdout.splitlines()
        assert len(lines) == len(calls)
        return lines

    return run


def draws(seed, count, sizes):
    rng = random.Random(seed)

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    for _ in range(count):
        nx, ny, n = (log(*s) for s in sizes)
        yield (rng.randrange(1, 6), rng.choice([FORWARD, FORWARD, FORWARD_F64, BACKWARD]), nx, ny,
               n, rng.random() < 0.8)


# All sizes that the entry points take, the usual ones, and the largest holograms.
@pytest.mark.parametrize("seed,sizes", [(1, [(1, 1 << 20), (1, 1 << 20), (1, 4000000)]),
                                        (2, [(1, 4096), (1, 4096), (1, 100000)]),
                                        (3, [(1 << 17, 1 << 20), (1 << 14, 1 << 19), (1, 3000)])])
def test_plans_stay_in_their_bounds(plans, seed, sizes):
    calls = list(draws(seed, 15000, sizes))
    checked = 0
    for c, line in zip(calls, plans(calls)):
        _, op, nx, ny, n, _ = c
        size = int(line.split("bytes ")[1].split()[0])
        if size + nx * ny * (8 if op == FORWARD_F64 else 4) + 16 * n > HBM:
            continue  # (no such call fits the memory)
        assert "bad" not in line, (c, line)
        checked += 1
    assert checked > 3000


# What the parity tests of these sizes exercise.
@pytest.mark.parametrize("call,route", [
    ((COMPENSATED, FORWARD, 333, 197, 337), "one-launch"),
    ((COMPENSATED, FORWARD, 365, 339, 10048), "direct-form"),
    ((COMPENSATED, FORWARD, 64, 48, 128), "one-launch"),
    ((COMPENSATED, FORWARD, 64, 48, 129), "direct-form"),
    ((COMPENSATED, FORWARD, 700, 500, 9001), "tiles shape 0 slices 9 passes 1 "),
    ((COMPENSATED, FORWARD, 1920, 1080, 65537), "tiles shape 1 slices 1 passes 3 "),
    ((COMPENSATED, FORWARD, 1100, 1500, 65001), "tiles shape 0 slices 2 passes 2 "),
    ((COMPENSATED, FORWARD, 4100, 2113, 9), "tiles shape 0 slices 1 passes 1 "),
    ((F16X3, FORWARD, 64, 48, 1025), "tiles shape 6 "),
    ((F16X3, FORWARD, 400, 300, 4901), "tiles shape 3 slices 6 passes 1 "),
    ((SEPARABLE, FORWARD, 256, 200, 12001), "tiles shape 5 slices 13 passes 1 "),
    ((SEPARABLE, FORWARD, 3840, 2160, 64), "tiles shape 0 "),
    ((F16, FORWARD, 6029, 4883, 9), "tiles shape 0 "),
    ((F16, FORWARD, 640, 480, 90001), "tiles shape 1 slices 6 passes 3 "),
    ((BF16, FORWARD, 1382, 471, 36661), "tiles shape 2 slices 4 passes 2 "),
    ((BF16, FORWARD, 3839, 2159, 200), "tiles shape 0 "),
])
def test_routes_of_the_parity_tests(plans, call, route):
    line, = plans([call + (1,)])
    assert line.startswith(route), line
