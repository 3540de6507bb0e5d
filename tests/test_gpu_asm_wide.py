"""The additive Schwarz overlap sum by plain loads, the form of meshes whose planes of
boxes exceed a 2 GiB buffer window, forced on small ones (SEM_ASM_WIDE=1): the same
values in the same order as the windowed form, bit for bit (p = 2, where a node lies in
up to 27 boxes, and above), and against the oracle; both precisions, boundary-condition
mixes, single elements in a direction."""
import numpy as np
import pytest

from pairs import Pair, host, rel_err
from paper_2110_07663_amd import sem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [sem.F64, sem.F32])
@pytest.mark.parametrize("p,shape,bc", [
    (2, (3, 4, 3), (1, 0, 1, 1, 0, 0)), (2, (1, 3, 2), (0,) * 6), (3, (3, 2, 3), (1,) * 6),
    (7, (2, 1, 3), (0, 1, 1, 0, 1, 0)), (10, (1, 2, 2), (1,) * 6)])
def test_plain_loads(monkeypatch, prec, p, shape, bc):
    t = __import__("torch")
    out = []
    for wide in ("0", "1"):
        monkeypatch.setenv("SEM_ASM_WIDE", wide)
        P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother="asm", bc=bc, smoother_prec=prec,
                 lambda_override=[2.0], oracle=wide == "1")
        r, ro = P.random_local(31)
        out.append(host(P.gpu.apply_S(r.to(t.float64 if prec == sem.F64 else t.float32))))
    np.testing.assert_array_equal(*out)
    assert rel_err(out[1], P.ora.levels[0].apply_S(ro)) < (1e-12 if prec == sem.F64 else 1e-5)
