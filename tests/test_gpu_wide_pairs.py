"""Cyclic reduction of link pairs of 17 to 64 rows: the factorization and the
solve against the FP64 oracle at the edges of its tile counts (17, 32, 33, 48,
49, 64 rows), at one to many pairs (no reduction level, odd and even counts)
and with borders of zero to four tiles with and without global rows.

Tolerance: the same elimination in another order, so FP64 rounding times the
conditioning of these well-scaled points (x, z in [0.1, 2], delta = 1e-4): the
1e-10 of the other direction tests.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401

SHAPES = [
    dict(N=2, m=(70, 90), n="2m", l=(33, 33), n0=0),            # a single pair
    dict(N=3, m=(70, 90), n="2m", l=(17, 64), n0=3),            # two pairs of different tile counts
    dict(N=4, m=(70, 90), n="2m", l=(48, 49), n0=17, ng=2),     # three
    dict(N=9, m=(66, 80), n="2m", l=(2, 48), n0=0, ng=5),       # eight, three tiles, global rows alone
    dict(N=18, m=(66, 80), n="2m", l=(33, 48), n0=48, ng=16),   # seventeen, a border of four tiles
    dict(N=34, m=(66, 70), n="2m", l=(49, 56), n0=24),          # thirty-three, four tiles
    dict(N=7, m=(40, 60), n="2m", l=(17, 32), n0=64),           # two tiles
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N{N}-l{l}-n0{n0}".format(**s).replace(" ", ""))
def test_wide_pairs(dev, shape):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(shape, density=0.3), 5)
    print("case", shape, flush=True)
    x, z, r = point(inst)
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    d1 = P.solve(*(T(v, dev) for v in r))[:3]
    f = newton.factor(inst, x, z, 1e-6, 1e-4)
    for a, b in zip(d1, newton.solve(f, *r)):
        assert rel(H(a), b) < 1e-10
    assert P.pivots() == 0
    d2 = P.solve_noalloc(*(T(v, dev) for v in r))[:3]
    for a, b in zip(d1, d2):
        assert np.array_equal(H(a), H(b))
    P.close()


def test_two_workspaces_side_by_side(dev):  # noqa: F811
    """A solve in the handle's workspace and one in the static workspace, on two
    streams at a time, leave what they leave one after the other."""
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(SHAPES[5], density=0.3), 5)
    print("case", SHAPES[5], flush=True)
    x, z, r = point(inst)
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    ra, rb = [T(v, dev) for v in r], [T(-2.0 * v, dev) for v in r]
    wa = [H(v) for v in P.solve(*ra)[:3]]
    wb = [H(v) for v in P.solve_noalloc(*rb)[:3]]
    torch.cuda.synchronize()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(10):
        da = P.solve(*ra, stream=sa)[:3]
        db = P.solve_noalloc(*rb, stream=sb)[:3]
        torch.cuda.synchronize()
        for got, want in zip((*da, *db), wa + wb):
            assert np.array_equal(H(got), want)
    P.close()
