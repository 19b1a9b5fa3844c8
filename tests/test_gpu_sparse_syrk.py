"""The block SYRK over nonzero lists against the dense one: bitwise equal factors,
both precisions, at ragged rows, columns and stages (64 columns), at the edges of
the column groups (128 rows), rows without and with many nonzeros, blocks of both
kinds side by side.  Each problem is large enough for the lists to be chosen in
both precisions (two work items per CU, 20 us to gain).

The fused launch mode multiplies the dense tiles of the same blocks, so the
factors of the other modes must be equal to its to the bit.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, dev, point  # noqa: E402, F401

CASES = [
    (dict(N=520, m=(145, 160), n="2m", l=(2, 9), n0=5), 0.05),
    (dict(N=700, m=(113, 128), n=256, l=3, n0=0), 0.08),
    (dict(N=570, m=(113, 128), n=193, l=3, n0=1), 0.03),
    (dict(N=90, m=(250, 310), n=640, l=5, n0=3), 0.02),
    (dict(N=340, m=(10, 300), n="2m", l=(1, 6), n0=2), 0.1),     # small blocks keep the dense tiles
    (dict(N=36, m=(600, 660), n="2m", l=2, n0=2), 0.02),
]


@pytest.mark.parametrize("shape,dens", CASES)
def test_bitwise(dev, shape, dens):  # noqa: F811
    from paper_2412_07731_amd.ahlp import FP32_REFINE, Problem
    print("case", shape, dens, flush=True)
    inst = gen.generate(dict(shape, density=dens), 11)
    rng = np.random.default_rng(1)
    a = inst.A[-1]
    a[1, :] = np.where(rng.random(a.shape[1]) < 0.6, 0.5, 0.0)   # a row of many nonzeros
    a[2, 1:] = 0.0                                               # one of a single one
    a[2, 0] = 1.0
    x, z, _ = point(inst)
    P = Problem(inst)
    some = sorted({0, 1, inst.N // 3, inst.N // 2, inst.N - 2, inst.N - 1})
    for prec in (0, FP32_REFINE):
        P.set_launch(mode="fused")
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
        ref = [P.debug_block(i) for i in some]
        for mode in ("batched", "per_block"):
            P.set_launch(mode=mode)
            P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
            for i, r in zip(some, ref):
                for u, v in zip(P.debug_block(i), r):
                    assert np.array_equal(u, v), (prec, mode, i)
    P.close()
