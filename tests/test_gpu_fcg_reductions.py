"""The FCG and PCG iterations against the oracle: (p, A p) from the element shares of
every order, A p read before its gather-scatter (SEM_GS_ZDEFER=0: after it), and the
sums closed by the last block (few blocks) or by a second launch (past 64 blocks of 512
values: 32768 nodes of all elements), for odd and even node counts."""
import numpy as np
import pytest

from pairs import Pair, dev, host, rel_err
from paper_2110_07663_amd import sem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zdefer", ["1", "0"])
@pytest.mark.parametrize("krylov", [sem.KRYLOV_FCG, sem.KRYLOV_PCG])
@pytest.mark.parametrize("p,shape,bc", [
    (1, (3, 3, 3), (1,) * 6), (2, (3, 1, 3), (1,) * 6), (4, (3, 3, 1), (0, 1, 1, 0, 0, 0)),
    (6, (2, 3, 3), (1, 0, 0, 1, 0, 1)), (7, (4, 4, 4), (1,) * 6), (7, (5, 4, 4), (1,) * 6),
    (9, (1, 2, 2), (1,) * 6), (10, (2, 2, 1), (1,) * 6), (3, (8, 9, 8), (1,) * 6)])
def test_fixed_iterations(monkeypatch, zdefer, krylov, p, shape, bc):
    monkeypatch.setenv("SEM_GS_ZDEFER", zdefer)
    name = {sem.KRYLOV_FCG: "fcg", sem.KRYLOV_PCG: "pcg"}[krylov]
    sched = (p, 1) if p > 1 else (1,)
    P = Pair(shape, p, mesh="sin", schedule=sched, smoother="jacobi", krylov=krylov, bc=bc,
             lambda_override=[1.6], coarse="dense")
    f = lambda X: np.sin(3 * X[0]) * np.cos(2 * X[1]) + X[2]
    xg, info = P.gpu.solve(P.gpu.rhs(dev(f(host(P.gpu.coords(0))))), rtol=1e-30, maxit=4, allow_noconv=True)
    res = P.ora.solve(P.ora.rhs(f(P.ora.fine.X)), tol=1e-30, maxit=4, krylov=name)
    assert info.iters == res.iters
    assert rel_err(host(xg), res.x) < 1e-11


def test_solution_vector_on_8_bytes():
    t = __import__("torch")
    P = Pair((8, 4, 5), 7, mesh="sin", schedule=(7, 1), smoother="jacobi", lambda_override=[1.6],
             coarse="dense", oracle=False)  # past one launch: the update takes the x and y steps
    b, _ = P.random_local(5)
    pad = t.zeros(b.numel() + 1, dtype=t.float64, device="cuda")
    x, _ = P.gpu.solve(b, rtol=1e-30, maxit=3, allow_noconv=True)
    y, _ = P.gpu.solve(b, x=pad[1:], rtol=1e-30, maxit=3, allow_noconv=True)
    assert rel_err(host(y), host(x).reshape(-1)) < 1e-12
