"""The autotuner ranks tiles by what a frame runs: under its tile a frame takes no
more than an eighth longer than under the best of all candidates.  (Tiles ranked
by another path's launches were up to 1.28 times the best here; the shorter of
several frames of a fixed number of iterations differs by 2-3%.)"""
import itertools
import time

import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

pytestmark = pytest.mark.gpu


def _frame_s(bp):
    bp.plan(2)
    best = np.inf
    for _ in range(6):
        t = time.perf_counter()
        bp.plan(6)
        best = min(best, (time.perf_counter() - t) / 6)
    return best


@pytest.mark.parametrize("n,G,N,W,rects", [(1, 8, 32, 20, 4), (16, 8, 32, 20, 4), (256, 8, 32, 20, 4), (1, 8, 170, 20, 30)])
def test_tuned_frame_is_near_the_best(n, G, N, W, rects):
    from paper_2308_10169_amd import sepso
    maps = [I.dynamic_map(i % 16, S=366.0, n_static=rects // 3, n_moving=rects - rects // 3, side=(8.0, 30.0))
            for i in range(n)]
    sws = [I.dynamic_swarm(m.scale, seed=8, instance=i, groups=G, particles=N, waypoints=W, iters=40, at_mode=0)
           for i, m in enumerate(maps)]
    print(f"autotune n={n} {G}x{N}x{W} rects={rects}", flush=True)
    times = {}

    def add(tune):
        bp = sepso.BatchPlanner(maps, sws, tune=tune)
        times[tune] = min(times.get(tune, np.inf), _frame_s(bp))
        bp.close()

    for tune in itertools.product((4, 8, 12, 16, 24), (64, 128, 256)):
        if tune[0] * tune[1] <= 4096:
            add(tune)
    bp = sepso.BatchPlanner(maps, sws)
    tune = bp.autotune()
    bp.close()
    best = min(times, key=times.get)
    for _ in range(3):  # the two in turn, so that a slow spell of the host meets both
        add(best)
        add(tune)
    print(f"tuned {tune} {times[tune] * 1e6:.0f} us, best {best} {times[best] * 1e6:.0f} us",
          flush=True)
    assert times[tune] <= 1.125 * times[best]
