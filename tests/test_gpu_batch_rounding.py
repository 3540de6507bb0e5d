"""Right sides of one problem solved together and one at a time on levels where the
boundary nodes of all of them exceed the limit of the one-launch gather-scatter and
those of one do not: the updates sum a node's copies in the same order, so the
iterates agree bit for bit (degrees whose vectors fit 16 and 8 bytes, and an odd
number of nodes, both precisions)."""
import numpy as np
import pytest

from pairs import dev, host
from paper_2110_07663_amd import sem
from paper_2110_07663_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p,sched,sm,prec,nrhs", [
    (8, 7, (7, 3, 1), sem.SMOOTH_RAS, sem.F32, 4), (8, 9, (9, 5, 1), sem.SMOOTH_RAS, sem.F32, 2),
    (8, 5, (5, 3, 1), sem.SMOOTH_JACOBI, sem.F64, 4), (7, 6, (6, 3, 1), sem.SMOOTH_JACOBI, sem.F64, 4)])
def test_joint_equals_in_turn(monkeypatch, n, p, sched, sm, prec, nrhs):
    t = __import__("torch")
    opts = sem.make_opts(schedule=sched, smoother=sm, smoother_prec=prec, batch_rhs=nrhs)
    S = sem.Solver(n, n, n, wl.sampled_mesh(n, n, n, sem.gll_nodes(p)[0], wl.sin_map(0.05)), p, p,
                   opts=opts)
    X = host(S.coords(0))
    bs = [S.rhs(dev(wl.sinusoid(1 + k, 1, 2 + k % 2)[0](X[0], X[1], X[2]))) for k in range(nrhs)]
    out = {}
    for mode in ("1", "0"):
        monkeypatch.setenv("SEM_BATCH_JOINT", mode)
        xs = [t.zeros_like(b) for b in bs]
        sem.batch_solve([S], [bs], [xs], rtol=1e-8, maxit=100)
        out[mode] = [host(x) for x in xs]
    for a, b in zip(out["1"], out["0"]):
        np.testing.assert_array_equal(a, b)
