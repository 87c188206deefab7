"""The learned initializer's products where their tiles change: row counts that
take each of the kernels, rows and k-steps past a tile's or a step's end.

Forward rows are independent: sampled rows (the first, the last and those
around tile edges) against the FP64 oracle, which rounds to BF16 at the same
points, with the tolerances of test_gpu_learned.  Gradients of a large batch
against the mean of its parts' (the same products at other sizes; FP32
summation order and a rare BF16 rounding boundary differ)."""
import numpy as np
import pytest

from oracle import pyorc as orc

from test_gpu_learned import SIZES, _cos, _inputs, _rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    from paper_2308_10169_amd import sepso
    sepso.lib()
    return sepso


@pytest.mark.parametrize("rows", [1, 33, 520, 1100, 2570, 5130])
def test_forward_rows(sp, rows):
    print(f"forward rows={rows}", flush=True)
    lin = sp.LearnedInit(max_rows=(rows + 31) // 32 * 32, seed=7)
    W, b = sp.split_params(lin.get_weights().astype(np.float64))
    x, _ = _inputs(rows, 6)
    y = lin.forward(x)
    idx = sorted({i for i in (0, 15, 16, 31, 32, 63, 64, 127, 128, rows // 2, rows - 2, rows - 1) if 0 <= i < rows})
    ref = orc.mlp(SIZES, W, b, x[idx].astype(np.float64), round=True, grads=False)["y"]
    for i, r in zip(idx, ref):
        assert _rel(y[i], r) <= 1e-2 and _cos(y[i], r) >= 0.999, (i, _rel(y[i], r))
    lin.close()


# 96 rows: three k-steps (a last one of half the width); 4128: 129 k-steps on
# 128 x 128 tiles and 64 x 128 forward tiles, parts of 43 k-steps on 64 x 64
@pytest.mark.parametrize("rows,parts", [(96, 3), (4128, 3)])
def test_gradients_of_parts(sp, rows, parts):
    print(f"gradients rows={rows}", flush=True)
    lin = sp.LearnedInit(max_rows=rows, seed=8)
    x, t = _inputs(rows, 12)
    n = rows // parts
    loss, g = lin.grads(x, t)
    got = [lin.grads(x[i:i + n], t[i:i + n]) for i in range(0, rows, n)]
    assert abs(loss - np.mean([p[0] for p in got])) <= 1e-5 * loss
    gW, gb = sp.split_params(g.astype(np.float64))
    qW, qb = sp.split_params(sum(p[1].astype(np.float64) for p in got) / parts)
    for l in range(4):
        for a, want in ((gW[l], qW[l]), (gb[l], qb[l])):
            # the loss scale 2 / (B n) is rounded, and dY with it to BF16: a
            # third is no power of two, so each side's dY differs by up to one
            # BF16 step, 2^-8, at random over its 320 B values; chains of four
            # such roundings average out over rows to well below 1e-2
            assert _rel(a, want) <= 1e-2 and _cos(a, want) >= 0.9999, (l, _rel(a, want), _cos(a, want))
    lin.close()
