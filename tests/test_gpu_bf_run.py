"""The whole-run benchmark-function kernel where its plan changes: one to
three particles per lane group, rows on 1 to 64 lanes, fewer random-factor
sets ahead than lanes, more than eight groups, and a move owed at the start of
a call.  Bit-identical to the two-launch path (same operations, same order)."""
import numpy as np
import pytest

from paper_2308_10169_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("func", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", [(8, 20, 30), (5, 8, 137), (4, 7, 256), (16, 40, 8), (12, 30, 18), (9, 91, 3)])
def test_run_plans(func, shape):
    from paper_2308_10169_amd import sepso as sp
    G, N, D = shape
    S = 2
    hy = np.tile(I.HYPER8[np.arange(G) % 8], (S, 1))
    print(f"bf run func={func} shape={shape}", flush=True)
    a = sp.BFSwarm(func, G, N, D, 60, hy, seed=9, swarms=S)
    b = sp.BFSwarm(func, G, N, D, 60, hy, seed=9, swarms=S, stepwise=True)
    for n in (9, 1, 30):
        a.step(n)
        b.step(n)
        sa, sb = a.get_state(), b.get_state()
        for k in ("X", "V", "P", "f", "Pf", "gbest_n", "gbest_f"):
            assert np.array_equal(sa[k], sb[k]), (n, k)
        assert (sa["k"], sa["ctr"], sa["pending"]) == (sb["k"], sb["ctr"], sb["pending"])
    sa["pending"] = 1  # the next call starts with the move
    a.set_state(sa)
    b.set_state(sa)
    a.step(4)
    b.step(4)
    sa, sb = a.get_state(), b.get_state()
    for k in ("X", "V", "P", "f", "Pf", "gbest_n", "gbest_f"):
        assert np.array_equal(sa[k], sb[k]), k
    a.close()
    b.close()
