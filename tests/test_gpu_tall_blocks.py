"""The block factorization of tall blocks (a launch per panel of four tile
columns) against the FP64 oracle: every remainder of the last panel, ragged
last tiles, bordered rows of none to several tiles, blocks of different heights
in one launch, and many more blocks than fit one row per wave.

Tolerances: L and W as in the stage parity test (1e-12 and 1e-11, FP64 rounding
of a factorization of up to 720 rows; componentwise growth m eps = 2e-13); FP32
factors within m_i eps_32 times the row scale, 4 x 720 x 6e-8 = 2e-4.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401

SHAPES = [
    dict(N=1, m=641, n=1282, l=0, n0=0),               # 41 tile columns, no border
    dict(N=2, m=(656, 672), n="2m", l=5, n0=3),        # 41 and 42
    dict(N=3, m=(673, 720), n="2m", l=(1, 20), n0=40),  # 43 to 45, borders of several tiles
    dict(N=3, m=(100, 700), n="2m", l=(2, 9), n0=4),   # beside panel blocks
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N{N}-m{m}-l{l}-n0{n0}".format(**s).replace(" ", ""))
def test_tall_factor(dev, shape):  # noqa: F811
    from paper_2412_07731_amd.ahlp import FP32_REFINE, Problem
    inst = gen.generate(dict(shape, density=0.1), 2)
    print("case", shape, flush=True)
    x, z, r = point(inst)
    f = newton.factor(inst, x, z, 1e-6, 1e-4)
    P = Problem(inst)
    for prec, tl, tw, td in ((0, 1e-12, 1e-11, 1e-10), (FP32_REFINE, 2e-4, 2e-4, None)):
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
        d = P.solve(*(T(v, dev) for v in r))[:3]
        for i in range(inst.N):
            L, W = P.debug_block(i)
            assert rel(L, f.L[i]) < tl, ("L", i)
            if f.W[i].size:
                assert rel(W, f.W[i]) < tw, ("W", i)
        assert P.pivots() == 0
        if td:
            for a, b in zip(d, newton.solve(f, *r)):
                assert rel(H(a), b) < td
    # one block at a time, and again: bitwise the same factors
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    a = [P.debug_block(i) for i in range(inst.N)]
    P.set_launch(per_block=True)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    for i in range(inst.N):
        for u, v in zip(a[i], P.debug_block(i)):
            assert np.array_equal(u, v)
    P.close()
