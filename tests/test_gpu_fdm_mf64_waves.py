"""The FP64 Schwarz local solves on the matrix cores with one and with four wavefronts
per element (SEM_FDM_MF64_WAVES; by default four up to 640 elements and one above, from
p = 7 on) against the oracle: RAS and ASM, every degree with both forms, element counts
that fill the last workgroup of four and that do not, boundary-condition mixes, and the
residual form inside the smoother."""
import numpy as np
import pytest

from pairs import Pair, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", ["1", "4"])
@pytest.mark.parametrize("smoother", ["ras", "asm"])
@pytest.mark.parametrize("p,shape,bc", [
    (7, (3, 2, 2), (1,) * 6), (8, (3, 3, 1), (0, 1, 1, 0, 1, 1)), (9, (2, 3, 1), (1, 0, 0, 1, 0, 1)),
    (9, (2, 2, 2), (1,) * 6), (10, (1, 2, 3), (1, 1, 0, 1, 0, 0)), (10, (5, 1, 1), (1,) * 6)])
def test_waves_per_element(monkeypatch, waves, smoother, p, shape, bc):
    monkeypatch.setenv("SEM_FDM_MF64_WAVES", waves)
    P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother=smoother, bc=bc, lambda_override=[2.0])
    g, o = P.random_local(51)
    zg, zo = host(P.gpu.apply_S(g)), P.ora.levels[0].apply_S(o).reshape(-1)
    assert rel_err(zg, zo) < 1e-12
    assert np.abs(zg - zo).max() < 1e-12 * np.abs(zo).max()
    b, bo = P.random_local(52)
    P.gpu.smooth(b, g, level=0)
    assert rel_err(host(g), P.ora.smooth(bo, o, level=0)) < 1e-12
