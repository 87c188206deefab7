"""The launch that ends a frame of one-launch iterations: its first block writes
the control block while the instance's other blocks may only start, and all of
them leave the swarm as the last iteration left it.  Launches of hundreds of
blocks, one instance whose frame ends early and many that end in different
launches, several times over; every instance's whole state bit for bit against
the instance alone, stepped (two launches an iteration, nothing written beside
readers)."""
import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

pytestmark = pytest.mark.gpu
KEYS = ("X", "V", "P", "f", "L", "Pf", "PL", "Q", "PQ", "gbest_n", "gbest_f", "hyper")


@pytest.mark.parametrize("n_inst,G,N,W,tune,T", [(1, 8, 1700, 64, (4, 256), 40), (30, 8, 170, 20, (4, 256), 45),
                                                 (60, 8, 256, 11, (12, 256), 60)])
def test_every_block_ends_with_the_frame(n_inst, G, N, W, tune, T):
    from paper_2308_10169_amd import sepso
    maps = [I.dynamic_map(70 + i, S=300.0, n_static=40, n_moving=20, side=(4.0, 15.0)) for i in range(n_inst)]
    sws = [I.dynamic_swarm(m.scale, seed=9, instance=i, groups=G, particles=N, waypoints=W, iters=T - i % 7,
                           at_mode=2 if i % 2 == 0 else 0,
                           hsef_every=4 if n_inst == 1 else 10) for i, m in enumerate(maps)]
    print(f"one launch end n={n_inst} {G}x{N}x{W} tune={tune}", flush=True)
    ref = []
    for m, sw in zip(maps, sws):
        one = sepso.Planner(m, sw)
        one.set_tune(*tune)
        one.step_frame(T)
        ref.append(one.get_state())
        one.close()
    for _ in range(3):
        bp = sepso.BatchPlanner(maps, sws, tune=tune)
        r = bp.plan(1)
        for i, sb in enumerate(ref):
            sa = bp.get_state(i)
            for k in KEYS:
                assert np.array_equal(sa[k], sb[k]), (i, k)
            assert (sa["tbest"], sa["k"], sa["ctr"]) == (sb["tbest"], sb["k"], sb["ctr"]), i
            assert r["iters"][0, i] == sb["k"] and r["cost"][0, i] == sb["tbest"][2], i
        bp.close()
