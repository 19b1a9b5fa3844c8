"""The reduction of the Schur complement in groups of link pairs against the FP64
oracle, at the edges of its rule: as many pairs as one group takes and one more,
the first counts with two and three stages, with borders of no, one, two and four
tiles, with and without global rows, and a border alone.

Tolerance: the same elimination with its sums in another order, so FP64 rounding
times the conditioning of these well-scaled points (x, z in [0.1, 2], delta =
1e-4): the 1e-10 of the other direction tests.
"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401

ONE = dict(m=(10, 14), n="2m", l=(1, 5))
SHAPES = [dict(ONE, N=N, n0=n0, ng=ng) for N, n0, ng in [
    (1, 7, 0), (1, 40, 3),                            # no pair
    (2, 0, 0), (3, 16, 0), (17, 16, 1), (17, 0, 0),   # one group of at most 16
    (18, 16, 0), (18, 0, 0), (258, 3, 0),             # a stage more
    (2, 17, 0), (9, 17, 0), (9, 55, 9),               # one group of at most 8
    (10, 32, 0), (10, 33, 2), (66, 60, 0),            # a stage more
    (300, 5, 2), (90, 48, 0), (600, 20, 4),           # two stages, two, three
]]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N{N}-n0{n0}-ng{ng}".format(**s))
def test_schur_factor(dev, shape):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(shape, density=0.3), 12)
    print("case", shape, flush=True)
    x, z, r = point(inst)
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    d = P.solve(*(T(v, dev) for v in r))[:3]
    f = newton.factor(inst, x, z, 1e-6, 1e-4)
    for a, b in zip(d, newton.solve(f, *r)):
        assert rel(H(a), b) < 1e-10
    assert P.pivots() == 0
    P.close()
