"""The exact coarse solve with its planes in blocks (SEM_COARSE_PLANES) against the
oracle's dense solve, inside a V-cycle: one block for the whole grid, two, three
(the middle block alone between the chains) and more, with a last block of fewer
planes, Dirichlet and mixed faces, and several right sides through the batched
solve's shared sweeps."""
import pytest

from pairs import Pair, host, rel_err
from paper_2110_07663_amd import sem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("planes", ["1", "2", "3", "4", "6", "7", None])
@pytest.mark.parametrize("shape,bc", [((3, 2, 6), (1,) * 6), ((5, 6, 6), (1, 0, 0, 1, 1, 0))])
def test_vcycle_with_blocks_of_planes(monkeypatch, planes, shape, bc):
    if planes:
        monkeypatch.setenv("SEM_COARSE_PLANES", planes)
    for prec, tol in ((sem.F64, 1e-12), (sem.F32, 1e-5)):
        P = Pair(shape, 3, mesh="sin", schedule=(3, 1), smoother="ras", bc=bc, smoother_prec=prec,
                 lambda_override=[1.8], coarse="dense")
        r, ro = P.random_local(81)
        assert rel_err(host(P.gpu.vcycle(r)), P.ora.vcycle(ro)) < tol


@pytest.mark.parametrize("planes", ["2", "3", "7"])
def test_right_sides_share_the_sweeps(monkeypatch, planes):
    t = __import__("torch")
    monkeypatch.setenv("SEM_COARSE_PLANES", planes)
    o = sem.make_opts(schedule=(3, 1), smoother=sem.SMOOTH_RAS, smoother_prec=sem.F32, batch_rhs=3)
    from paper_2110_07663_amd import workloads as wl
    s = sem.Solver(3, 2, 6, wl.box_vertices(3, 2, 6), 1, 3, opts=o)
    g = t.Generator(device="cuda").manual_seed(3)
    b = []
    for _ in range(3):
        u = t.rand(s.levels[0].nglobal, generator=g, device="cuda", dtype=t.float64)
        b.append(s.apply_A(s.gather(u)))
    joint = [t.zeros_like(v) for v in b]
    sem.batch_solve([s], [b], [joint], rtol=1e-10)
    monkeypatch.setenv("SEM_BATCH_JOINT", "0")  # the right sides one at a time
    alone = [t.zeros_like(v) for v in b]
    sem.batch_solve([s], [b], [alone], rtol=1e-10)
    for x, y in zip(joint, alone):
        assert t.equal(x, y)
