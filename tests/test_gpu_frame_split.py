"""Frames of one workgroup per instance where a particle's update is shared by
several threads and each iteration's random factors are drawn by themselves:
the factors cross waves, so every thread has to wait for them.  That is so for
a batch of unlike swarms (one that fills more than half the workgroup's
threads beside one that does not) and for swarms that fill a CU's LDS.  Bit for
bit against each instance alone, stepped iteration by iteration (two launches
each, the same operations in the same order)."""
import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

KEYS = ("X", "V", "P", "f", "L", "Pf", "PL", "Q", "PQ", "gbest_n", "gbest_f", "hyper")
# (groups, particles, waypoints) of each instance, rectangles, tile
CASES = [
    ([(4, 32, 8), (8, 40, 8)], 3, (8, 256)), ([(4, 32, 8), (8, 40, 8)] * 3, 3, (4, 64)),
    ([(8, 32, 10), (8, 40, 10)], 2, (8, 256)), ([(4, 32, 8), (8, 40, 8)], 1, (12, 256)),
    ([(1, 9, 4), (8, 47, 8)], 1, (4, 256)), ([(4, 47, 32)], 2, (8, 128)),
    ([(1, 101, 62)], 1, (12, 256)), ([(4, 32, 48)] * 64, 2, (4, 256))]


def split(shapes, K, B):
    """Threads per particle of each instance, and iterations whose factors are
    drawn together: the smallest instance share, halved until the swarm fits
    LDS (the library's rule, for the tiles and sizes above)."""
    def ppb(W, R):
        return max(2, (B // R // ((W + K) // K)) & ~1)

    R = 1
    while 2 * R <= B // 64 and sum(-(-G * N // ppb(W, 2 * R)) for G, N, W in shapes) <= 512:
        R *= 2
    blocks = max(-(-G * N // ppb(W, R)) for G, N, W in shapes)
    T = min(blocks * (B // R), 512 // (B // R) * (B // R))
    parts = [max(1, T // (G * N)) for G, N, W in shapes]
    ahead = min(parts + [8])

    def lds(a):
        return max(4 * ((3 * G * N + G + 1) * 2 * (W | 1) + (7 + 3 * a) * G * N + 9 * G + 64 + 2 * T + 4)
                   for G, N, W in shapes)
    while ahead > 1 and lds(ahead) > 159 * 1024:
        ahead //= 2
    return parts, ahead


@pytest.mark.parametrize("shapes,n,tune", CASES)
def test_cases_share_a_particle_without_drawing_ahead(shapes, n, tune):
    parts, ahead = split(shapes, *tune)
    assert ahead == 1 and max(parts) > 1


@pytest.mark.gpu
@pytest.mark.parametrize("shapes,n,tune", CASES)
def test_frame_equals_instances_stepped(shapes, n, tune):
    from paper_2308_10169_amd import sepso
    T = 30
    maps = [I.dynamic_map(40 + i, S=150.0, n_static=1, n_moving=n - 1, side=(5.0, 25.0)) for i in range(len(shapes))]
    sws = [I.dynamic_swarm(m.scale, seed=8, instance=i, groups=G, particles=N, waypoints=W, iters=T, at_mode=2,
                           hsef_every=7) for i, (m, (G, N, W)) in enumerate(zip(maps, shapes))]
    print(f"frame split shapes={shapes[:2]} x {len(shapes)} n={n} tune={tune}", flush=True)
    bp = sepso.BatchPlanner(maps, sws, tune=tune)
    r = bp.plan(1)
    for i in range(0, len(shapes), max(1, len(shapes) // 8)):
        m, sw = maps[i], sws[i]
        one = sepso.Planner(m, sw)
        one.set_tune(*tune)
        one.step_frame(T)
        sa, sb = bp.get_state(i), one.get_state()
        for k in KEYS:
            assert np.array_equal(sa[k], sb[k]), (i, k)
        assert (sa["tbest"], sa["k"], sa["ctr"]) == (sb["tbest"], sb["k"], sb["ctr"]), i
        assert r["cost"][0, i] == sb["tbest"][2] and r["iters"][0, i] == sb["k"], i
        one.close()
    bp.close()
