"""The Schur solve in groups of link pairs against the FP64 oracle, at the edges
of its rule: as many pairs as the last stage takes and one more, the first
counts with two and three stages, each tile count of the pairs, one and two
positions a wave (borders of up to and over two tiles) and no border.

Tolerance: the same elimination with its sums in another order, so FP64 rounding
times the conditioning of these well-scaled points (x, z in [0.1, 2], delta =
1e-4): the 1e-10 of the other direction tests.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401

ONE = dict(m=(10, 14), n="2m", l=(1, 5))
SHAPES = [
    dict(ONE, N=2, n0=5),
    dict(ONE, N=33, n0=5),                # the last stage full (32 pairs)
    dict(ONE, N=34, n0=5, ng=2),          # a stage before it
    dict(ONE, N=66, n0=0),                # no border
    dict(ONE, N=1026, n0=32),             # two stages
    dict(ONE, N=17, n0=40),               # one position a wave: full, a stage, two stages
    dict(ONE, N=18, n0=64, ng=9),
    dict(ONE, N=258, n0=33),
    dict(N=9, m=(40, 50), n="2m", l=(17, 24), n0=7),     # two tiles: full, a stage, two stages
    dict(N=10, m=(40, 50), n="2m", l=(2, 24), n0=50),
    dict(N=67, m=(40, 50), n="2m", l=(17, 20), n0=3, ng=1),
    dict(N=5, m=(70, 80), n="2m", l=(33, 40), n0=7),     # three
    dict(N=6, m=(70, 80), n="2m", l=(5, 40), n0=50),
    dict(N=18, m=(70, 80), n="2m", l=(33, 36), n0=0),
    dict(N=3, m=(100, 110), n="2m", l=(49, 50), n0=20),  # four
    dict(N=4, m=(100, 110), n="2m", l=(4, 50), n0=0),
    dict(N=10, m=(100, 110), n="2m", l=(49, 50), n0=20, ng=4),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N{N}-l{l}-n0{n0}".format(**s).replace(" ", ""))
def test_schur_solve(dev, shape):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(shape, density=0.3), 11)
    print("case", shape, flush=True)
    x, z, r = point(inst)
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    d1 = P.solve(*(T(v, dev) for v in r))[:3]
    f = newton.factor(inst, x, z, 1e-6, 1e-4)
    for a, b in zip(d1, newton.solve(f, *r)):
        assert rel(H(a), b) < 1e-10
    d2 = P.solve_noalloc(*(T(v, dev) for v in r))[:3]
    for a, b in zip(d1, d2):
        assert np.array_equal(H(a), H(b))
    P.close()
