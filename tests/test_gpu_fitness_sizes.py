"""sepso_fitness at the sizes where its kernel changes course: polygons of 1
to 33 and more edges (the per-lane and the whole-wave walk), maps beyond one
LDS pass of vertices or polygons and a polygon beyond one by itself, few and
many segments (one or two per thread, one or more rounds per block), and
axis-parallel and zero-length segments.  Against the FP64 oracle: counts
equal where it flags no degenerate test, else inside its bracket; lengths and
fitness within FP32 rounding of at most 65 summed terms (1e-5 relative)."""
import math

import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I
from test_gpu_fitness import _gpu, _paths, check

pytestmark = pytest.mark.gpu
S = 256.0


def _ngon(m, cx, cy, r):
    th = np.arange(m) * (2.0 * math.pi / m) + 0.1
    return np.stack([cx + r * np.cos(th), cy + r * np.sin(th)], axis=1)


def _map(case):
    rng = np.random.default_rng(3)
    rects = list(I.random_rects(rng, S, S, 900 if case == "polys" else 24, 2.0, 9.0))
    polys = {"rects": rects[:5], "polys": rects,
             "edges": rects + [_ngon(m, 20 + 22 * k, 128.0, 30.0) for k, m in enumerate((3, 5, 31, 32, 33, 64, 100))],
             "verts": rects[:9] + [_ngon(3000, 90.0, 140.0, 60.0)] + rects[9:] + [_ngon(2561, 170.0, 120.0, 50.0)]}
    return I.make_map(S, S, polys[case], (3.0, 5.0), (250.0, 251.0))


@pytest.mark.parametrize("case,n,W", [("rects", 1, 1), ("rects", 131075, 1), ("edges", 257, 31),
                                      ("edges", 130, 42), ("edges", 4100, 64), ("verts", 65, 63), ("polys", 70, 20)])
def test_fitness_sizes(case, n, W):
    sepso = _gpu()
    spec = _map(case)
    rng = np.random.default_rng(n + W)
    X = _paths(rng, spec, n, W)
    if case == "edges":  # a third of the paths on a coarse grid: axis-parallel and zero-length segments
        X[::3] = np.round(X[::3] / 32.0) * 32.0
    print(f"fitness sizes case={case} n={n} W={W} edges={spec.n_edges}", flush=True)
    out = sepso.fitness(spec, X, W, 30.0, 4)
    keep = np.arange(n) if n <= 300 else rng.choice(n, 300, replace=False)
    check(spec, X[keep], W, 30.0, 4, {k: v[keep] for k, v in out.items()})
    # what lies outside the sample: the same path gives the same result wherever it stands in the call
    again = sepso.fitness(spec, X[::-1].copy(), W, 30.0, 4)
    for k in ("f", "L", "Q"):
        assert np.array_equal(out[k], again[k][::-1]), k
