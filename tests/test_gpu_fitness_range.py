"""sepso_fitness on coordinates at the ends of a float's range: the counts are
those of testing every segment against every edge with the same FP32
operations, also where their products overflow.  The reference makes each fused
multiply-add from an exact product and sum in extended precision (a 48-bit
product and a 64-bit sum: no second rounding that could change a sign here)."""
import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

E, F = np.longdouble, np.float32


def _fma(a, b, c):
    with np.errstate(all="ignore"):
        return (E(a) * E(b) + E(c)).astype(F)


def _count(verts, ends, X, W):
    """Crossings of every path with quads of four vertices each."""
    n = len(X)
    pts = np.empty((n, W + 2, 2), F)
    pts[:, 0], pts[:, -1] = ends[0], ends[1]
    pts[:, 1:-1, 0], pts[:, 1:-1, 1] = X[:, :W], X[:, W:]
    p, q = pts[:, :-1, None, :], pts[:, 1:, None, :]
    a = verts[None, None]
    b = np.roll(verts.reshape(-1, 4, 2), -1, axis=1).reshape(-1, 2)[None, None]
    with np.errstate(all="ignore"):
        d, e = q - p, b - a
        nc = _fma(d[..., 1], p[..., 0], -(d[..., 0] * p[..., 1]))
        ce = _fma(e[..., 0], a[..., 1], -(e[..., 1] * a[..., 0]))

        def line(v):  # the segment's line
            return _fma(d[..., 0], v[..., 1], _fma(-d[..., 1], v[..., 0], nc))

        def edge(v):
            return _fma(e[..., 0], v[..., 1], _fma(-e[..., 1], v[..., 0], -ce))

        def opposite(x, y):
            return ((x < 0) & (y > 0)) | ((x > 0) & (y < 0))

        return (opposite(line(a), line(b)) & opposite(edge(p), edge(q))).sum(axis=(1, 2))


def _case(scale):
    rng = np.random.default_rng(4)
    n, W, polys = 200, 6, 30
    X = (rng.uniform(0.0, 1.0, (n, 2 * W)) * scale).astype(F)
    c = rng.uniform(0.0, 1.0, (polys, 1, 2))
    h = 10.0 ** rng.uniform(-3.0, -0.3, (polys, 1, 1))
    verts = ((c + h * rng.uniform(-1.0, 1.0, (polys, 4, 2))) * scale).astype(F).reshape(-1, 2)
    ends = (np.array([[0.02, 0.03], [0.97, 0.95]]) * scale).astype(F)
    return X, verts, ends, W


def test_reference_counts_as_the_oracle():
    from oracle import pyorc as orc
    X, verts, ends, W = _case(4096.0)
    X, verts, ends = np.round(X), np.round(verts), np.round(ends)  # the maps' grid holds whole numbers
    spec = I.make_map(4096.0, 4096.0, list(verts.reshape(-1, 4, 2)), ends[0], ends[1])
    r = orc.fitness(orc.Map(spec), X.astype(np.float64), W, 1.0, 1)
    clean = r["n_deg"] == 0
    assert clean.sum() > 100 and np.array_equal(_count(verts, ends, X, W)[clean], r["Q"][clean])


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1e-15, 1.0, 1e9, 4e18, 2e19, 4e19, 6.3e19, 1e20, 1e30])
def test_counts_at_any_scale(scale):
    import ctypes as C

    import torch
    from paper_2308_10169_amd import sepso
    X, verts, ends, W = _case(scale)
    n = len(X)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda()
           for x in (np.arange(0, len(verts) + 1, 4, dtype=np.int32), verts, ends, X)]
    f, L = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    Q = torch.zeros(n, dtype=torch.int32, device="cuda")
    ptr = [C.c_void_p(x.data_ptr()) for x in dev]
    print(f"fitness range scale={scale}", flush=True)
    sepso._check(sepso.lib().sepso_fitness_noalloc(len(verts) // 4, len(verts), *ptr, n, W, 1.0, 1,
                                                   *[C.c_void_p(x.data_ptr()) for x in (f, L, Q)],
                                                   C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    assert np.array_equal(Q.cpu().numpy(), _count(verts, ends, X, W))
