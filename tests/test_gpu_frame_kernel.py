"""A frame planned in one launch (one workgroup per instance) against the same
frame stepped iteration by iteration (two launches each): the swarm, the
bests, the control state and the online outer swarm bit for bit (the same
operations in the same order).  Shapes with one pass and several passes of
blocks, more particles than threads, tiles that deal the rectangles over wave
groups, rows of odd and single waypoints, convex polygons, every Auto
Truncation mode."""
import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

pytestmark = pytest.mark.gpu
KEYS = ("X", "V", "P", "f", "L", "Pf", "PL", "Q", "PQ", "gbest_n", "gbest_f", "hyper")


def _scene(kind, n):
    if kind == "convex":
        return I.convex_map(n, n_rects=1, n_convex=2)
    return I.dynamic_map(n, S=150.0, n_static=1, n_moving=n - 1, side=(5.0, 25.0))


@pytest.mark.parametrize("G,N,W,scene,n,tune,at,hsef,T", [
    (4, 32, 8, "rects", 4, None, 0, 0, 30), (8, 32, 20, "rects", 4, (12, 256), 2, 10, 50),
    (8, 32, 20, "rects", 2, (4, 64), 1, 3, 25), (1, 1, 1, "rects", 1, None, 3, 2, 9),
    (3, 33, 7, "rects", 3, (8, 128), 3, 4, 70), (2, 300, 3, "rects", 2, (4, 256), 2, 5, 20),
    (8, 24, 10, "convex", 5, (8, 64), 0, 5, 20), (60, 4, 9, "rects", 3, (8, 256), 1, 7, 30)])
def test_frame_kernel_equals_launches(G, N, W, scene, n, tune, at, hsef, T):
    from paper_2308_10169_amd import sepso
    spec = _scene(scene, n)
    sw = I.dynamic_swarm(spec.scale, seed=5, groups=G, particles=N, waypoints=W, iters=T, at_mode=at, hsef_every=hsef)
    print(f"frame kernel G={G} N={N} W={W} {scene} n={n} tune={tune}", flush=True)
    a, b = sepso.Planner(spec, sw), sepso.Planner(spec, sw)
    if tune:
        a.set_tune(*tune)
        b.set_tune(*tune)
    r = a.plan_frame()
    b.step_frame(T)
    sa, sb = a.get_state(), b.get_state()
    for k in KEYS:
        assert np.array_equal(sa[k], sb[k]), k
    assert (sa["tbest"], sa["k"], sa["ctr"]) == (sb["tbest"], sb["k"], sb["ctr"])
    assert r["iters"] == sb["k"] and r["cost"] == sb["tbest"][2]
    oa, ob = a.get_outer(), b.get_outer()
    for k in oa:
        assert np.array_equal(oa[k], ob[k]), k
    a.close()
    b.close()
