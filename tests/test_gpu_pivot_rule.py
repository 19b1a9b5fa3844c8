"""Replaced pivots in every kernel that factorizes: rows of zeros (without
regularization, so their pivots are exactly zero) at the edges of tiles and of the tile
factor's panels of four columns, several in one tile and a whole tile of them, in
blocks of each block-factor kernel's heights, in link pairs of one to four tiles, in
the first, a middle and the last pair, and in the border's global rows.

The count is exact.  Directions: the 1e-10 of the other direction tests (rows of zeros
drop out, and the remaining M_i = A D A' of well-scaled points have condition numbers
of some 1e2).  FP32 factors: W within 4 m eps_32 of its scale, 2e-4 at most, as for the
regularized ones; its rows of replaced pivots are zero.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from oracle import newton  # noqa: E402
from paper_2412_07731_amd import gen  # noqa: E402
from tests.test_gpu_parity import T, H, dev, point, rel  # noqa: E402, F401


def instance(cfg, rows=(), links=(), glob=()):
    """rows: (block, rows), links: (pair, link rows), glob: global rows, all zeroed"""
    inst = gen.generate(dict(cfg, density=0.3), 9)
    for i, rr in rows:
        inst.A[i] = inst.A[i].copy()
        inst.C[i] = inst.C[i].copy()
        inst.A[i][list(rr)] = 0.0
        inst.C[i][list(rr)] = 0.0
    for j, rr in links:
        inst.FR[j], inst.FL[j] = inst.FR[j].copy(), inst.FL[j].copy()
        inst.FR[j][list(rr)] = 0.0
        inst.FL[j][list(rr)] = 0.0
    for k in glob:
        inst.Wg = [w.copy() for w in inst.Wg]
        for w in inst.Wg:
            w[k] = 0.0
        inst.Wg0 = inst.Wg0.copy()
        inst.Wg0[k] = 0.0
    return inst, sum(len(list(r)) for _, r in (*rows, *links)) + len(glob)


def check(dev, inst, replaced, fp32=False):
    from paper_2412_07731_amd.ahlp import FP32_REFINE, Problem
    x, z, r = point(inst)
    f = newton.factor(inst, x, z, 0.0, 0.0)
    assert f.pivots == replaced
    P = Problem(inst)
    P.factor(T(x, dev), T(z, dev), 0.0, 0.0)
    d = P.solve(*(T(v, dev) for v in r))[:3]
    assert P.pivots() == replaced
    for a, b in zip(d, newton.solve(f, *r)):
        assert rel(H(a), b) < 1e-10
    if fp32:
        P.factor(T(x, dev), T(z, dev), 0.0, 0.0, precision=FP32_REFINE)
        assert P.pivots() == replaced
        for i in range(inst.N):
            assert rel(P.debug_block(i)[1], f.W[i]) < 2e-4
    P.close()


ROWS = [(0,), (15,), (3, 4), (17, 18, 30), range(32, 48), (0, 31, 63, 64)]
BLOCKS = [
    (dict(N=3, m=[70, 66, 80], n="2m", l=3, n0=2), "panel, 2 rows a wave"),
    (dict(N=3, m=[200, 250, 240], n="2m", l=3, n0=2), "panel, 5"),
    (dict(N=2, m=[345, 350], n="2m", l=3, n0=2), "panel, 6"),
    (dict(N=2, m=[420, 560], n="2m", l=3, n0=2), "panel of eight waves"),
    (dict(N=2, m=[660, 700], n="2m", l=3, n0=2), "tall"),
]


@pytest.mark.parametrize("rows", ROWS, ids=lambda r: "-".join(map(str, list(r)[:4])))
@pytest.mark.parametrize("cfg,name", BLOCKS, ids=[n.replace(" ", "") for _, n in BLOCKS])
def test_block_rows(dev, cfg, name, rows):  # noqa: F811
    print("case", name, list(rows), flush=True)
    m = cfg["m"]
    last = [m[1] - 1 - r for r in rows] if len(rows) < 16 else [m[1] - 1]   # counted from the last row
    inst, k = instance(cfg, rows=[(0, rows), (1, last)])
    check(dev, inst, k, fp32=True)


LINKS = [
    (dict(N=6, m=40, n="2m", l=12, n0=3), [(0, (0,)), (2, (3, 4, 11)), (4, (11,))]),        # one tile, one group
    (dict(N=40, m=30, n="2m", l=16, n0=20), [(0, (15,)), (16, (0, 7)), (31, range(16)), (38, (2,))]),   # stages
    (dict(N=5, m=70, n="2m", l=30, n0=3), [(0, (0, 17)), (2, (15, 16, 29)), (3, range(16, 30))]),       # two tiles
    (dict(N=5, m=90, n="2m", l=45, n0=3), [(1, (0, 31, 32, 44)), (3, (40,))]),               # three
    (dict(N=5, m=120, n="2m", l=60, n0=3), [(1, (0, 20, 33, 59)), (2, range(48, 60))]),      # four
]


@pytest.mark.parametrize("cfg,links", LINKS, ids=["l%d-N%d" % (c["l"], c["N"]) for c, _ in LINKS])
def test_link_rows(dev, cfg, links):  # noqa: F811
    print("case", cfg, flush=True)
    check(dev, *instance(cfg, links=links))


@pytest.mark.parametrize("l,n0,ng,glob", [
    (4, 6, 3, (0,)), (4, 6, 3, (1, 2)), (4, 20, 18, (0, 15, 16, 17)), (12, 30, 30, (3, 20, 29)),
    (20, 6, 3, (2,)), (40, 20, 18, (0, 16)),
])
def test_global_rows(dev, l, n0, ng, glob):  # noqa: F811
    print("case", l, n0, ng, glob, flush=True)
    check(dev, *instance(dict(N=6, m=60, n="2m", l=l, n0=n0, ng=ng), glob=glob))


def test_all_at_once(dev):  # noqa: F811
    inst, k = instance(dict(N=6, m=[60, 300, 60, 700, 60, 60], n="2m", l=20, n0=6, ng=3),
                       rows=[(1, (5, 6)), (3, (0, 699))], links=[(2, (0, 19))], glob=(1,))
    print("case", k, flush=True)
    check(dev, inst, k)
