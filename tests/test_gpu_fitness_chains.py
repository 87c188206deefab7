"""sepso_fitness on polygons of many edges, which the kernel cuts into chains:
lengths at which the last chain is short, full or a single edge, long polygons
between short ones, several in one LDS pass, and polygons that exceed a pass by
themselves (one, two in a row, ending at a pass's edge).  Against the FP64
oracle as in test_gpu_fitness.py: counts equal where it flags no degenerate
test, else inside its bracket."""
import math

import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I
from test_gpu_fitness import _gpu, _paths, check

pytestmark = pytest.mark.gpu
S = 256.0


def _ring(m, cx, cy, r, teeth):
    """m vertices around (cx, cy); with teeth every second one is further in."""
    th = np.arange(m) * (2.0 * math.pi / m) + 0.1
    rr = r * np.where(np.arange(m) % 2, 1.0 - teeth, 1.0)
    return np.stack([cx + rr * np.cos(th), cy + rr * np.sin(th)], axis=1)


def _map(lengths, teeth):
    rng = np.random.default_rng(len(lengths))
    polys = []
    for i, m in enumerate(lengths):
        polys.append(_ring(m, *rng.uniform(60.0, 196.0, 2), rng.uniform(10.0, 55.0), teeth))
        polys += list(I.random_rects(rng, S, S, i % 3, 2.0, 9.0))
    return I.make_map(S, S, polys, (3.0, 5.0), (250.0, 251.0))


@pytest.mark.parametrize("teeth", [0.0, 0.4])
@pytest.mark.parametrize("lengths,n,W", [
    ((33, 34, 62, 63, 64, 65, 93, 94, 95), 70, 20), ((33,) * 70, 300, 7), ((125,) * 20, 130, 31), ((1240, 1241), 65, 5),
    ((2559,), 65, 3), ((2560,), 65, 3), ((2561,), 40, 63), ((5119,), 40, 12), ((5118, 7, 2600, 2700, 33), 33, 9),
    ((40, 8000, 40), 64, 1), ((33, 64, 100), 4200, 64), ((3000, 50), 90000, 2)])
def test_long_polygons(lengths, n, W, teeth):
    sepso = _gpu()
    spec = _map(lengths, teeth)
    X = _paths(np.random.default_rng(n + W), spec, n, W)
    print(f"fitness chains {lengths[:4]} x {len(lengths)} n={n} W={W} teeth={teeth}", flush=True)
    out = sepso.fitness(spec, X, W, 30.0, 4)
    keep = np.arange(n) if n <= 300 else np.random.default_rng(1).choice(n, 200, replace=False)
    check(spec, X[keep], W, 30.0, 4, {k: v[keep] for k, v in out.items()})
    again = sepso.fitness(spec, X[::-1].copy(), W, 30.0, 4)
    for k in ("f", "L", "Q"):
        assert np.array_equal(out[k], again[k][::-1]), k
