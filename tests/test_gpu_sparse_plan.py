"""The problems that the tests of the compressed passes and of the nonzero-list SYRK
compare forms on do take those forms, in both precisions; and the SYRK's forms agree to
the bit on problems well inside the rule, so that a change of its constants does not
leave FP32, or blocks of both kinds side by side, untested.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests import test_gpu_sparse_passes, test_gpu_sparse_syrk  # noqa: E402
from tests.test_gpu_parity import H, T, dev, point, rel  # noqa: E402, F401


@pytest.mark.parametrize("k", range(len(test_gpu_sparse_syrk.CASES)))
def test_syrk_cases_are_on_lists(dev, k):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    shape, dens = test_gpu_sparse_syrk.CASES[k]
    P = Problem(gen.generate(dict(shape, density=dens), 11))
    _, a, b = P.debug_plan()
    print("case", shape, dens, a, b, flush=True)
    assert a > 0 and b > 0
    if k == 4:   # the one with small blocks
        assert a < shape["N"] and b < shape["N"]
    P.close()


@pytest.mark.parametrize("k", range(len(test_gpu_sparse_passes.CASES)))
def test_pass_cases_are_compressed(dev, k):  # noqa: F811
    """(at 50% nonzeros as well: up to 0.9 of the dense bytes, padding included)"""
    from paper_2412_07731_amd.ahlp import Problem
    shape, dens = test_gpu_sparse_passes.CASES[k]
    inst = gen.generate(dict(shape, density=dens), 3)
    inst.A[0][:, 1] = 0.0
    inst.A[1][3, :] = inst.A[1][3, :] + 0.25
    P = Problem(inst)
    print("case", shape, dens, P.debug_plan(), flush=True)
    assert P.debug_plan()[0]
    P.close()


@pytest.mark.parametrize("dens,compressed", [(0.5, True), (0.9, False)])
def test_directions_of_both_passes(dev, dens, compressed):  # noqa: F811
    """The same shape on both sides of the rule against the oracle (1e-10 as there)."""
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(N=4, m=(60, 140), n="2m", l=(2, 20), n0=5, ng=2, density=dens), 3)
    x, z, r = point(inst)
    P = Problem(inst)
    print("case", dens, P.debug_plan(), flush=True)
    assert P.debug_plan()[0] == compressed
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    d = P.solve(*(T(v, dev) for v in r))[:3]
    for a, b in zip(d, newton.solve(newton.factor(inst, x, z, 1e-6, 1e-4), *r)):
        assert rel(H(a), b) < 1e-10
    P.close()


def test_agreeing_lp_takes_both(dev):  # noqa: F811
    """test_ipm_sparse_and_dense_blocks_agree's two forms of one LP."""
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(N=6, m=(40, 70), n="2m", l=(2, 9), n0=6, density=0.1), 7)
    P = Problem(inst)
    inst.A = [np.where(a == 0.0, 1e-300, a) for a in inst.A]
    Q = Problem(inst)
    assert P.debug_plan()[0] and not Q.debug_plan()[0]
    P.close(), Q.close()


@pytest.mark.parametrize("shape,dens,both", [
    (dict(N=1100, m=(145, 160), n="2m", l=(2, 9), n0=5), 0.05, False),
    (dict(N=700, m=(10, 300), n="2m", l=(1, 6), n0=2), 0.08, True),
])
def test_bitwise_well_inside(dev, shape, dens, both):  # noqa: F811
    from paper_2412_07731_amd.ahlp import FP32_REFINE, Problem
    inst = gen.generate(dict(shape, density=dens), 11)
    x, z, _ = point(inst)
    P = Problem(inst)
    print("case", shape, dens, P.debug_plan(), flush=True)
    for lists in P.debug_plan()[1:]:
        assert inst.N // 4 < lists <= inst.N and (lists < inst.N) == both
    some = list(range(0, inst.N, inst.N // 12))
    for prec in (0, FP32_REFINE):
        P.set_launch(mode="fused")
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
        ref = [P.debug_block(i) for i in some]
        P.set_launch(mode="batched")
        P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4, precision=prec)
        for i, r in zip(some, ref):
            for u, v in zip(P.debug_block(i), r):
                assert np.array_equal(u, v), (prec, i)
    P.close()
