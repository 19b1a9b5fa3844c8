"""The row and column passes over the compressed blocks against the passes over
the dense tiles and the FP64 oracle: densities on both sides of the rule that
chooses between them, empty rows and columns, ragged tiles, with and without x_0
columns, rows of very different length.

A refined solve exercises every form (row passes with one vector, with and
without x_0, the column pass with its modes), an interior-point run those with
two and three.  Tolerance: the same products in another order, FP64 rounding of
sums of at most 600 terms on well-scaled points: the 1e-10 of the direction tests.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import ipm as oipm, lp, newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401

CASES = [
    (dict(N=3, m=17, n=35, l=4, n0=1), 0.05),
    (dict(N=5, m=(30, 70), n="2m", l=(1, 9), n0=17), 0.08),
    (dict(N=2, m=150, n=300, l=3, n0=0), 0.02),
    (dict(N=4, m=(60, 140), n="2m", l=(2, 20), n0=5, ng=2), 0.2),
    (dict(N=4, m=(60, 140), n="2m", l=(2, 20), n0=5, ng=2), 0.5),   # dense tiles
]


@pytest.mark.parametrize("shape,dens", CASES)
def test_directions(dev, shape, dens):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(shape, density=dens), 3)
    inst.A[0][:, 1] = 0.0            # an empty column
    inst.A[1][3, :] = inst.A[1][3, :] + 0.25   # a full row beside sparse ones
    print("case", shape, dens, flush=True)
    x, z, r = point(inst)
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 1e-6, 1e-4)
    d = P.solve(*(T(v, dev) for v in r))[:3]
    for a, b in zip(d, newton.solve(newton.factor(inst, x, z, 1e-6, 1e-4), *r)):
        assert rel(H(a), b) < 1e-10
    # refined on the unregularized system (rank deficient in the first case):
    # the oracle's backward error, as in the trajectory tests
    be = P.solve(*(T(v, dev) for v in r), max_refine=5, refine_tol=1e-14)[3]
    f = newton.factor(inst, x, z, 1e-6, 1e-4)
    rows, cols = lp.abs_row_col_sums(inst)
    opts = oipm.Options(max_refine=5, refine_tol=1e-14)
    _, eta = oipm.solve_refined(inst, f, r, lp.kkt_inf_norm(rows, cols, x, z), opts,
                                dict(refine=0, bkerr=0.0))
    assert be <= max(1e-12, 10 * eta)
    P.close()


def test_ipm_sparse_and_dense_blocks_agree(dev):  # noqa: F811
    """The same LP with its blocks above and below the rule: zeros replaced by
    1e-300 make every entry a nonzero without changing any product."""
    from paper_2412_07731_amd.ahlp import Problem
    inst = gen.generate(dict(N=6, m=(40, 70), n="2m", l=(2, 9), n0=6, density=0.1), 7)
    P = Problem(inst)
    x, y, z, res = P.ipm()
    full = gen.generate(dict(N=6, m=(40, 70), n="2m", l=(2, 9), n0=6, density=0.1), 7)
    full.A = [np.where(a == 0.0, 1e-300, a) for a in full.A]
    Q = Problem(full)
    x2, y2, z2, res2 = Q.ipm()
    o = oipm.solve(inst)
    assert res["iterations"] == res2["iterations"] == o.iterations
    assert abs(res["primal_obj"] - res2["primal_obj"]) <= 1e-8 * abs(res["primal_obj"])
    assert rel(H(x), H(x2)) < 1e-6
    P.close(), Q.close()
