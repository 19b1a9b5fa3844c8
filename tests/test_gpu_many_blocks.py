"""More blocks than a grid has rows (65535): tuning times every block-factor kernel on
all of them, the tall ones with a grid row per block, and the factorization after it
solves the system.

Blocks of one row and two columns without links, so the direction has a closed form:
FP64 rounding of a dozen operations on values in [0.1, 2], 1e-13 of the largest.
"""
from types import SimpleNamespace

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from tests.test_gpu_parity import T, H, dev, rel  # noqa: E402, F401


def test_autotune_of_many_blocks(dev):  # noqa: F811
    from paper_2412_07731_amd.ahlp import Problem
    N, delta, rho = 65537, 1e-4, 1e-6
    rng = np.random.default_rng(1)
    A = rng.uniform(0.5, 1.5, (N, 1, 2))
    none = np.zeros((0, 2))
    inst = SimpleNamespace(N=N, n0=0, m=np.ones(N, int), n=np.full(N, 2), l=np.zeros(N - 1, int), A=list(A),
                           C=[], FR=[none] * (N - 1), FL=[none] * (N - 1), F0=None, Wg=None, Wg0=None, ub=None,
                           b=np.ones(N), c=np.ones(2 * N))
    print("case", N, flush=True)
    P = Problem(inst)
    assert P.autotune() == 1
    x, z, rx, rz = (rng.uniform(0.1, 2.0, 2 * N) for _ in range(4))
    ry = rng.uniform(0.1, 2.0, N)
    P.factor(T(x, dev), T(z, dev), rho, delta)
    d = P.solve(T(rx, dev), T(ry, dev), T(rz, dev))[:3]
    D, h, a = 1.0 / (z / x + rho), rx - rz / x, A.reshape(N, 2)
    dy = (ry + (a * (D * h).reshape(N, 2)).sum(1)) / ((a * a * D.reshape(N, 2)).sum(1) + delta)
    dx = D * ((a * dy[:, None]).ravel() - h)
    for got, want in zip(d, (dx, dy, (rz - z * dx) / x)):
        assert rel(H(got), want) < 1e-13
    P.close()
