"""The block substitutions by size of the largest block (waves, rows a wave and
steps ahead follow from it).

With a border: against the FP64 oracle at both sides of each line of the rule.
Tolerance: the same sums in another order, FP64 rounding on well-scaled points: the
1e-10 of the direction tests.

Without one, blocks are independent and every sum of a block runs in the same order
under any choice, so a block's direction is bitwise the same beside a larger block,
with FP64 and with FP32 factors.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401

# largest blocks of 8, 9, 16, 17, 24, 25, 40, 41 and 72 tile rows (the middle one's
# border takes three)
MS = [5, 80, 81, 208, 209, 336, 337, 592, 593, 1104]


@pytest.mark.parametrize("m", MS)
def test_bordered(dev, m):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(N=3, m=[max(1, m // 3), m, max(1, m // 2 + 3)], n="2m", l=1, n0=5, density=0.3), 4)
    print("case", m, flush=True)
    x, z, r = point(inst)
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    d = P.solve(*(T(v, dev) for v in r))[:3]
    for a, b in zip(d, newton.solve(newton.factor(inst, x, z, 1e-6, 1e-4), *r)):
        assert rel(H(a), b) < 1e-10
    P.close()


@pytest.mark.parametrize("m,big", [(16, 129), (128, 257), (129, 385), (256, 640), (300, 1104), (640, 700)])
def test_beside_a_larger_block(dev, m, big):  # noqa: F811
    from paper_2412_07731_amd.ahlp import FP32_REFINE, Problem
    both = gen.generate(dict(N=2, m=[m, big], n="2m", l=0, n0=0, density=1.0), 8)
    one = gen.generate(dict(N=1, m=[m], n="2m", l=0, n0=0, density=1.0), 8)
    one.A[0] = both.A[0]
    n = one.A[0].shape[1]
    print("case", m, big, flush=True)
    x, z, r = point(both)
    P, Q = Problem(both), Problem(one)
    for prec in (0, FP32_REFINE):
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
        Q.factor(T(x[:n], dev), T(z[:n], dev), 1e-6, 1e-4, precision=prec)
        a = P.solve(*(T(v, dev) for v in r))[:3]
        b = Q.solve(T(r[0][:n], dev), T(r[1][:m], dev), T(r[2][:n], dev))[:3]
        for u, v in zip(a, b):
            assert np.array_equal(H(u)[:H(v).size], H(v))
    P.close(), Q.close()
