"""Additive Schwarz in FP32: the local solves on the matrix cores (the default
for 2 <= p <= 9) and on the vector pipe (SEM_FDM_MF32=0), and the overlap sum,
against the oracle for every degree (at p = 2 a node lies in up to 27 boxes,
else in up to 8), boundary-condition mixes and partly filled workgroups; inside
the smoother with A's deferred x and y steps taken as the box is read, the x
step alone, or neither (SEM_FDM_YSTEP, SEM_FDM_XSTEP)."""
import numpy as np
import pytest

from pairs import Pair, host, rel_err
from paper_2110_07663_amd import sem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mf32,xstep,ystep", [("1", "1", "1"), ("1", "1", "0"), ("1", "0", "1"),
                                              ("0", "1", "1")])
@pytest.mark.parametrize("p,shape,bc", [
    (2, (3, 3, 3), (1,) * 6), (2, (2, 3, 2), (0, 1, 1, 0, 0, 0)), (3, (3, 3, 2), (1, 0, 1, 1, 0, 1)),
    (4, (2, 3, 2), (0,) * 6), (5, (3, 2, 3), (1, 1, 0, 1, 1, 0)), (6, (2, 2, 2), (1,) * 6),
    (7, (4, 3, 2), (0, 1, 1, 0, 1, 1)), (7, (1, 1, 1), (1,) * 6), (8, (2, 2, 3), (1,) * 6),
    (9, (3, 2, 2), (0, 0, 1, 1, 0, 1)), (10, (2, 1, 2), (1,) * 6), (4, (1, 1, 1), (0,) * 6)])
def test_asm_fp32_forms(monkeypatch, mf32, xstep, ystep, p, shape, bc):
    t = __import__("torch")
    for k, v in (("MF32", mf32), ("XSTEP", xstep), ("YSTEP", ystep)):
        monkeypatch.setenv("SEM_FDM_" + k, v)
    P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother="asm", bc=bc, cheb_order=2,
             smoother_prec=sem.F32, lambda_override=[2.0])
    g, o = P.random_local(61)
    zg, zo = host(P.gpu.apply_S(g.to(t.float32))), P.ora.levels[0].apply_S(o).reshape(-1)
    assert rel_err(zg, zo) < 1e-5
    assert np.abs(zg - zo).max() < 1e-5 * np.abs(zo).max()
    b, bo = P.random_local(62)
    x = g.to(t.float32)
    P.gpu.smooth(b.to(t.float32), x, level=0)
    assert rel_err(host(x), P.ora.smooth(bo, o, level=0)) < 1e-5
