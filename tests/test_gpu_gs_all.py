"""The gather-scatter of all three directions in one launch (small levels by
default, SEM_GS_ALL=1 forces it) against the direction passes (SEM_GS_ALL=0):
the same sums in the same order, so every result agrees bit for bit, for the
operator, the Schwarz smoother, the smoothing step and the transfers, in both
precisions; degrees without interior nodes (p = 1), single elements in a
direction, and Dirichlet / Neumann mixes."""
import numpy as np
import pytest

from pairs import Pair, host, rel_err
from paper_2110_07663_amd import sem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("p,shape,bc", [
    (2, (3, 2, 2), (1,) * 6), (3, (1, 4, 1), (0,) * 6), (4, (2, 3, 5), (1, 0, 0, 1, 0, 0)),
    (5, (3, 3, 2), (0, 0, 1, 1, 0, 1)), (7, (4, 2, 3), (1,) * 6), (7, (8, 1, 2), (0, 1, 0, 0, 1, 0)),
    (9, (2, 2, 2), (0, 1, 1, 0, 1, 1))])
def test_one_launch_equals_the_passes(monkeypatch, prec, p, shape, bc):
    t = __import__("torch")
    dt = t.float64 if prec == "f64" else t.float32
    monkeypatch.setenv("SEM_GS_ZDEFER", "0")  # the updates read assembled vectors
    out = {}
    for form in ("0", "1"):
        monkeypatch.setenv("SEM_GS_ALL", form)
        P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother="ras", bc=bc, oracle=form == "1",
                 smoother_prec=sem.F64 if prec == "f64" else sem.F32, lambda_override=[2.0])
        g, o = P.random_local(71)
        b = P.random_local(72)[0].to(dt)
        x = g.to(dt)
        A = P.gpu.apply_A(x)
        if form == "1":
            assert rel_err(host(A), P.ora.levels[0].apply_A(o)) < (1e-12 if prec == "f64" else 1e-5)
        out[form] = [host(v) for v in (A, P.gpu.apply_S(x), P.gpu.restrict(x),
                                       P.gpu.smooth(b, x.clone()))]
    if prec == "f64":  # (in FP32 the passes let the x-face sums into the FDM's workgroups)
        for a, c in zip(out["0"], out["1"]):
            np.testing.assert_array_equal(a, c)
    else:
        for a, c in zip(out["0"][:3], out["1"][:3]):
            np.testing.assert_array_equal(a, c)
        assert rel_err(out["0"][3], out["1"][3]) < 1e-6
