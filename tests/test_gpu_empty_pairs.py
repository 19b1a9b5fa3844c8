"""Neighbouring blocks without link rows between them (l_j = 0) at the start, in the
middle and at the end of the chain, against the FP64 oracle: pairs of one tile in one
and in several stages of groups, wider pairs, a border over 64 columns, arrays that
end with their allocation.

Tolerance: the 1e-10 of the other direction tests (FP64 rounding on well-scaled
points); the empty pairs add no arithmetic.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401

M = [20, 24, 18, 30, 22]
CASES = [
    (M[:2], [0], 3, 0), (M[:2], [0], 0, 0), (M[:3], [0, 0], 17, 0),
    (M, [0, 4, 5, 3], 5, 0), (M, [4, 0, 0, 3], 5, 2), (M, [4, 5, 16, 0], 0, 0), (M, [0, 7, 0, 0], 40, 3),
    ([20] * 40, [0 if j % 3 else 9 for j in range(39)], 8, 0),          # two stages, most pairs empty
    ([20] * 300, [16] * 298 + [0], 32, 0),                              # whole pages, the last pair empty
    ([60] * 6, [0, 40, 0, 17, 0], 5, 2), ([60] * 6, [20, 0, 30, 0, 0], 20, 0),   # several tiles
    (M, [4, 0, 5, 0], 70, 0),                                           # a border over 64
]


@pytest.mark.parametrize("m,l,n0,ng", CASES, ids=lambda v: str(len(v)) if isinstance(v, list) else str(v))
def test_empty_pairs(dev, m, l, n0, ng):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    print("case", len(m), l[:8], n0, ng, flush=True)
    inst = gen.generate(dict(N=len(m), m=m, n="2m", l=l, n0=n0, ng=ng, density=0.3), 4)
    assert list(inst.l) == l
    x, z, r = point(inst)
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    d = P.solve(*(T(v, dev) for v in r))[:3]
    f = newton.factor(inst, x, z, 1e-6, 1e-4)
    for a, b in zip(d, newton.solve(f, *r)):
        assert rel(H(a), b) < 1e-10
    assert P.pivots() == 0
    for a, b in zip(d, P.solve_noalloc(*(T(v, dev) for v in r))[:3]):
        assert np.array_equal(H(a), H(b))
    P.close()
