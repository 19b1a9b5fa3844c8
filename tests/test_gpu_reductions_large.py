"""Reductions of 2^17 to over a million elements, at the edges of their split: the
objective values of an interior-point run, dot products over all of x and y on the
device, against the same products of the returned vectors.

Tolerance: sums of at most 1.1 million products in another order, in partial sums of at
most 4608 by 256 threads: far below 1e-11 of the sum of magnitudes.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import H, dev  # noqa: E402, F401


@pytest.mark.parametrize("n", [2048, 2049, 4096, 4097, 8192, 8193, 17000])
def test_objectives(dev, n):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(N=64, m=4, n=n, l=2, n0=0, density=0.05), 6)
    print("case", inst.n_tot, flush=True)
    P = Problem(inst)
    for _ in range(2):
        x, y, z, res = P.ipm(max_iter=3)
        xs, ys = H(x), H(y)
        assert abs(res["primal_obj"] - inst.c @ xs) <= 1e-11 * (np.abs(inst.c) @ np.abs(xs))
        assert abs(res["dual_obj"] - inst.b @ ys) <= 1e-11 * (np.abs(inst.b) @ np.abs(ys))
    P.close()
