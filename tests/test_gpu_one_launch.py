"""A frame whose iterations take one launch each (every block finds the bests
from all blocks' candidates) against the same frame stepped iteration by
iteration (two launches each): the swarm, the bests, the control state and the
online outer swarm bit for bit (the same operations in the same order), over
two frames.  Shapes with groups that span blocks and blocks that span groups,
one block, more candidates than two per thread, tiles that deal the rectangles
over wave groups, edge-by-edge polygons, every Auto Truncation mode, several
instances of different lengths.  (With 100 rectangles a swarm of any size here
is past the whole-frame kernel.)"""
import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

pytestmark = pytest.mark.gpu
KEYS = ("X", "V", "P", "f", "L", "Pf", "PL", "Q", "PQ", "gbest_n", "gbest_f", "hyper")


@pytest.mark.parametrize("G,N,W,n,tune,at,hsef,T", [
    (8, 170, 20, 30, (4, 256), 2, 10, 50), (3, 33, 7, 100, (8, 128), 1, 3, 40), (1, 1, 1, 100, None, 3, 2, 9),
    (60, 4, 9, 100, (8, 256), 0, 7, 30), (4, 640, 16, 100, (4, 64), 2, 0, 30), (2, 301, 31, 60, (12, 256), 0, 5, 12),
    (5, 50, 3, 100, (4, 64), 3, 1, 20)])
def test_one_launch_equals_two(G, N, W, n, tune, at, hsef, T):
    from paper_2308_10169_amd import sepso
    spec = I.dynamic_map(n, S=300.0, n_static=n // 2, n_moving=n - n // 2, side=(4.0, 15.0))
    sw = I.dynamic_swarm(spec.scale, seed=6, groups=G, particles=N, waypoints=W, iters=T, at_mode=at, hsef_every=hsef)
    print(f"one launch G={G} N={N} W={W} n={n} tune={tune}", flush=True)
    a, b = sepso.Planner(spec, sw), sepso.Planner(spec, sw)
    if tune:
        a.set_tune(*tune)
        b.set_tune(*tune)
    ra = a.plan_frame()
    b.step_frame(T)
    sa, sb = a.get_state(), b.get_state()
    for k in KEYS:
        assert np.array_equal(sa[k], sb[k]), k
    assert (sa["tbest"], sa["k"], sa["ctr"]) == (sb["tbest"], sb["k"], sb["ctr"])
    assert ra["iters"] == sb["k"] and ra["cost"] == sb["tbest"][2]
    oa, ob = a.get_outer(), b.get_outer()
    for k in oa:
        assert np.array_equal(oa[k], ob[k]), k
    a.close()
    b.close()


def test_instances_alone_and_together():
    # uneven instances: eight in one batch (one launch per iteration) and each
    # among 65 (which reserve no candidates: two launches), two frames
    from paper_2308_10169_amd import sepso
    maps, sws = [], []
    for i in range(65):
        m, shape = I.batch_instance(i, 3)
        maps.append(m)
        sws.append(I.dynamic_swarm(m.scale, seed=3, instance=i, **shape))
    few = sepso.BatchPlanner(maps[:8], sws[:8], tune=(4, 256))
    many = sepso.BatchPlanner(maps, sws, tune=(4, 256))
    for _ in range(2):
        rf, rm = few.plan(1, want_paths=True), many.plan(1, want_paths=True)
        for k in ("cost", "crossings", "iters", "truncated"):
            assert np.array_equal(rf[k], rm[k][:, :8]), k
        for i in range(8):
            assert np.array_equal(rf["paths"][i], rm["paths"][i]), i
    few.close()
    many.close()
