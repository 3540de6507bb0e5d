"""Chebyshev updates that read A's or S's output before its gather-scatter: all
steps on small levels (SEM_GS_ZDEFER=0: assembled there), the x and y steps on
others (SEM_GS_ALL=0; vectors that fit element rows), none (SEM_GS_XDEFER=0);
Jacobi smoothing scales on the way.  Against the oracle, for every order that has
its own update, odd and even N, boundary-condition mixes, one element in a
direction, zero and given starts (the V-cycle and the smoothing step), and
V-cycle vectors that overlap or are not 16-byte aligned."""
import numpy as np
import pytest

from pairs import Pair, host, rel_err
from paper_2110_07663_amd import sem

pytestmark = pytest.mark.gpu

FORMS = [{}, {"SEM_GS_ZDEFER": "0"}, {"SEM_GS_ALL": "0"},
         {"SEM_GS_ALL": "0", "SEM_GS_XDEFER": "0"}]


@pytest.mark.parametrize("form", range(len(FORMS)))
@pytest.mark.parametrize("smoother", ["jacobi", "ras"])
@pytest.mark.parametrize("p,shape,bc,order", [
    (3, (3, 2, 2), (1,) * 6, 2), (4, (2, 3, 1), (0, 1, 1, 0, 0, 0), 1), (5, (3, 3, 2), (0,) * 6, 3),
    (7, (4, 2, 3), (1, 0, 0, 1, 0, 1), 2), (7, (1, 1, 1), (1,) * 6, 2), (2, (3, 3, 3), (1,) * 6, 3)])
def test_updates_read_unassembled(monkeypatch, form, smoother, p, shape, bc, order):
    t = __import__("torch")
    for k, v in FORMS[form].items():
        monkeypatch.setenv(k, v)
    for prec, dt, tol in ((sem.F64, t.float64, 1e-12), (sem.F32, t.float32, 1e-5)):
        P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother=smoother, bc=bc, cheb_order=order,
                 smoother_prec=prec, lambda_override=[1.9], coarse="pcg")
        b, bo = P.random_local(91)
        x, xo = P.random_local(92)
        x = P.gpu.smooth(b.to(dt), x.to(dt))
        assert rel_err(host(x), P.ora.smooth(bo, xo, level=0)) < tol


@pytest.mark.parametrize("smoother", ["jacobi", "ras"])
def test_vcycle_vectors(monkeypatch, smoother):
    t = __import__("torch")
    P = Pair((3, 2, 4), 7, mesh="sin", schedule=(7, 3, 1), smoother=smoother,
             lambda_override=[1.9, 1.9], coarse="dense")
    r, ro = P.random_local(93)
    zo = P.ora.vcycle(ro)
    n = r.numel()
    assert rel_err(host(P.gpu.vcycle(r)), zo) < 1e-12
    pad = t.empty(2 * n + 2, dtype=t.float64, device="cuda")
    pad[1:n + 1] = r
    z = P.gpu.vcycle(pad[1:n + 1], out=pad[n + 1:2 * n + 1])  # 8-byte aligned
    assert rel_err(host(z), zo) < 1e-12
    assert t.equal(pad[1:n + 1], r)
    assert rel_err(host(P.gpu.vcycle(r, out=r)), zo) < 1e-12  # in place
