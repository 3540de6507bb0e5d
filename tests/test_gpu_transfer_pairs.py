"""Prolongation and restriction for every pair of degrees with compile-time sizes
and one without, against the oracle: partly filled workgroups, boundary-condition
mixes (the restriction forms the node weights from the grid position), and several
right sides through the V-cycle of a batched solve are covered by the batch tests."""
import pytest

from pairs import Pair, host, rel_err
from oracle import mg
from paper_2110_07663_amd import sem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pf,pc", [(2, 1), (3, 1), (3, 2), (4, 1), (4, 2), (5, 1), (5, 3), (6, 3),
                                   (7, 1), (7, 3), (7, 5), (8, 4), (9, 3), (9, 5), (9, 7), (10, 5),
                                   (10, 9)])
@pytest.mark.parametrize("shape,bc", [((3, 2, 3), (1, 0, 0, 1, 1, 0)), ((1, 5, 1), (0, 0, 1, 1, 0, 0))])
def test_transfers(pf, pc, shape, bc):
    t = __import__("torch")
    sched = (pf, pc) if pc == 1 else (pf, pc, 1)
    P = Pair(shape, pf, mesh="sin", schedule=sched, bc=bc, smoother_prec=sem.F32,
             lambda_override=[1.0] * 3)
    F, C = P.ora.levels[0], P.ora.levels[1]
    rf, rfo = P.random_local(101)
    xf, xfo = P.random_local(102, masked=False)
    xc, xco = P.random_local(103, level=1, masked=False)
    want_r = mg.restrict(F.num, C.num, F.J_to_coarse, rfo)
    want_p = xfo + mg.prolong(F.J_to_coarse, xco)
    for dt, tol in ((t.float64, 1e-12), (t.float32, 1e-6)):
        assert rel_err(host(P.gpu.restrict(rf.to(dt))), want_r) < tol
        assert rel_err(host(P.gpu.prolong(xc.to(dt), xf.clone().to(dt))), want_p) < tol
