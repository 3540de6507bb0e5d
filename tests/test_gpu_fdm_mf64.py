"""The FP64 Schwarz local solves on the matrix cores (v_mfma_f64_4x4x4, the
default for 2 <= p <= 10) and on the vector pipe (SEM_FDM_MF64=0) against the
oracle: RAS and ASM, every degree (lines and modes that fill their groups of
16 and 4, and that do not), partly filled workgroups, boundary-condition mixes,
a floating box, and the residual form r - rs inside the smoother."""
import numpy as np
import pytest

from pairs import Pair, host, rel_err

pytestmark = pytest.mark.gpu

CASES = [(2, (3, 2, 2), (1,) * 6), (3, (3, 3, 2), (1, 0, 1, 1, 0, 1)), (4, (2, 3, 2), (0,) * 6),
         (5, (3, 2, 3), (1, 1, 0, 1, 1, 0)), (6, (2, 2, 2), (1,) * 6),
         (7, (5, 3, 2), (0, 1, 1, 0, 1, 1)), (7, (1, 1, 1), (1,) * 6), (8, (2, 2, 3), (1,) * 6),
         (9, (3, 2, 2), (0, 0, 1, 1, 0, 1)), (10, (2, 1, 2), (1, 1, 1, 0, 1, 1)),
         # above 640 elements a wave solves a whole element also from p = 7 on
         (7, (9, 9, 8), (1, 1, 0, 1, 1, 0)),
         (4, (1, 1, 1), (0,) * 6)]  # a floating box: its constant mode is dropped


@pytest.mark.parametrize("mf64", ["1", "0"])
@pytest.mark.parametrize("smoother", ["ras", "asm"])
@pytest.mark.parametrize("p,shape,bc", CASES)
def test_fp64_local_solves(monkeypatch, mf64, smoother, p, shape, bc):
    monkeypatch.setenv("SEM_FDM_MF64", mf64)
    P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother=smoother, bc=bc,
             lambda_override=[2.0])
    g, o = P.random_local(51)
    zg, zo = host(P.gpu.apply_S(g)), P.ora.levels[0].apply_S(o).reshape(-1)
    assert rel_err(zg, zo) < 1e-12
    assert np.abs(zg - zo).max() < 1e-12 * np.abs(zo).max()
    b, bo = P.random_local(52)  # the post-smoothing residual formed as the box is read
    P.gpu.smooth(b, g, level=0)
    assert rel_err(host(g), P.ora.smooth(bo, o, level=0)) < 1e-12
