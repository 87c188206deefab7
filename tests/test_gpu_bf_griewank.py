"""Griewank's value near its optimum, where the cosines' product counts: one
launch per call against two launches per iteration on the same positions.
Equal bits where the rows are past 64 KiB three times over (or one lane holds a
whole row: its product has no last factor); below that the one-launch run
rounds the product by itself, so the values differ by at most that rounding
(half an ulp of a product up to 1: 2^-25) and the last one's (an ulp of the
larger value, where the two round apart)."""
import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 10, 30), (3, 5, 7), (5, 8, 64), (8, 20, 30), (12, 30, 18), (16, 40, 8),
                                   (5, 8, 137), (9, 91, 3)])
def test_paths_near_the_optimum(shape):
    from paper_2308_10169_amd import sepso as sp
    G, N, D = shape
    Q = (D + 3) // 4
    equal = D <= 4 or 16 * Q * (3 * G * N + G) + 28 * G * N + 40 * G > 65536
    hy = I.HYPER8[np.arange(G) % 8]
    print(f"griewank shape={shape} equal={equal}", flush=True)
    a, b = sp.BFSwarm(4, G, N, D, 60, hy, seed=3), sp.BFSwarm(4, G, N, D, 60, hy, seed=3, stepwise=True)
    st = a.get_state()
    rng = np.random.default_rng(D)
    st["X"] = (rng.standard_normal(st["X"].shape) * rng.choice([0.01, 0.1, 1.0], (*st["X"].shape[:-1], 1))).astype(np.float32)
    a.set_state(st)
    b.set_state(st)
    a.step(1)
    b.step(1)
    fa, fb = a.get_state()["f"].ravel(), b.get_state()["f"].ravel()
    if equal:
        assert np.array_equal(fa, fb)
    else:
        assert np.all(np.abs(fa.astype(np.float64) - fb) <= 2.0 ** -25 + np.spacing(np.maximum(fa, fb)))
    print(f"griewank differing values: {np.count_nonzero(fa != fb)} of {fa.size}", flush=True)
    a.close()
    b.close()
