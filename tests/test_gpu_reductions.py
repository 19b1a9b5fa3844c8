"""The reductions at the edges of their rule (one workgroup up to 1024 elements, a
workgroup per 1024, at most 64): an interior-point run's objective values, which
are dot products over all of x and y on the device, against the same products of
the returned vectors, twice on one handle (the arrival counts are back at zero).

Tolerance: sums of at most 70000 products in another order, 70000 x 1.1e-16 of the
sum of magnitudes at most: 1e-11 of it.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import H, dev  # noqa: E402, F401


@pytest.mark.parametrize("N,m,n,n0", [(1, 4, 8, 0), (2, 256, 512, 0), (2, 256, 512, 1), (9, 64, 128, 5),
                                      (64, 512, 1024, 0), (64, 512, 1024, 7)])
def test_objectives(dev, N, m, n, n0):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(N=N, m=m, n=n, l=min(4, m) if N > 1 else 0, n0=n0, density=0.02 if m > 100 else 0.3), 6)
    print("case", N, m, n, n0, flush=True)
    P = Problem(inst)
    for _ in range(2):
        x, y, z, res = P.ipm()
        xs, ys = H(x), H(y)
        c, b = inst.c, inst.b
        assert c.size == xs.size and b.size == ys.size
        assert abs(res["primal_obj"] - c @ xs) <= 1e-11 * (np.abs(c) @ np.abs(xs))
        assert abs(res["dual_obj"] - b @ ys) <= 1e-11 * (np.abs(b) @ np.abs(ys))
    P.close()
