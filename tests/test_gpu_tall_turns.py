"""Tall blocks by the dozen, whose workgroups take several groups of rows in turn:
to the bit the factors of launches with one block, where every group of rows has a
workgroup of its own."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, dev, point  # noqa: E402, F401


@pytest.mark.parametrize("N", [48, 140])
def test_turns(dev, N):  # noqa: F811
    from paper_2412_07731_amd.ahlp import FP32_REFINE, Problem
    inst = gen.generate(dict(N=N, m=(645, 680), n="2m", l=(1, 9), n0=3, density=0.02), 2)
    print("case", N, flush=True)
    x, z, _ = point(inst)
    P = Problem(inst)
    some = [0, 1, N // 2, N - 1]
    for prec in (0, FP32_REFINE):
        P.set_launch(per_block=False)
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
        a = [P.debug_block(i) for i in some]
        P.set_launch(per_block=True)
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
        for i, ref in zip(some, a):
            for u, v in zip(P.debug_block(i), ref):
                assert np.array_equal(u, v), (prec, i)
    P.close()
