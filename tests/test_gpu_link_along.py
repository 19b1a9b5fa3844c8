"""Link columns in the block SYRK's launch and in one of their own: the rule
between them goes by the number of work items (at most four a compute unit), so
the same blocks are factored on both sides of it and against the launch per
block, which has the gather of its own.

The values are those of the same gather and the same products: equality.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2412_07731_amd import gen  # noqa: E402
from paper_2412_07731_amd.ahlp import FP32_REFINE, FP64  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point  # noqa: E402, F401

# a block of 16 to 64 rows has one item of the SYRK's and one to three of the
# link columns', so that 200 blocks are below the 1024 of 256 units and 1025 above
SHAPES = [
    dict(N=2, m=(16, 16), n="2m", l=(2, 2), n0=0),               # more links than SYRK units
    dict(N=3, m=(17, 140), n="2m", l=(3, 16), n0=40, ng=3),      # ragged, several of each a block
    dict(N=9, m=(30, 64), n="2m", l=(1, 17), n0=5),
    dict(N=200, m=(16, 64), n="2m", l=(2, 6), n0=3),
    dict(N=1025, m=(16, 32), n="2m", l=(2, 6), n0=3),
]


@pytest.mark.parametrize("prec", [FP64, FP32_REFINE], ids=["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "N{N}-n0{n0}".format(**s))
def test_link_along(dev, shape, prec):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(shape, density=0.3), 3)
    print("case", shape, prec, flush=True)
    x, z, _ = point(inst)
    P = Problem(inst)
    got = []
    for per_block in (False, True):
        P.set_launch(per_block)
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, prec)
        got.append([P.debug_block(i) for i in (0, inst.N - 1)] + [P.debug_schur()])
    for a, b in zip(*got):
        for u, v in zip(a if isinstance(a, tuple) else (a,), b if isinstance(b, tuple) else (b,)):
            assert np.array_equal(u, v)
    P.close()
