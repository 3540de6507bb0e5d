"""The exact coarse solve on boxes so thin that a pivot of a block of planes falls below
the singularity test although the level is regular: factored again in single planes, it
stays exact (no CG iteration) and equals the factorisation that starts with single
planes; a singular level (Neumann everywhere) still goes to the CG."""
import pytest

from paper_2110_07663_amd import sem
from paper_2110_07663_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [sem.F64, sem.F32])
def test_thin_boxes_stay_exact(monkeypatch, prec):
    t = __import__("torch")
    xyz = wl.box_vertices(4, 4, 4)
    xyz[..., 2] *= 2e-7
    o = sem.make_opts(schedule=(3, 1), smoother_prec=prec, lambda_override=[2.6],
                      coarse_solver=sem.COARSE_DIRECT)
    out = []
    for planes in (None, "1"):
        if planes:
            monkeypatch.setenv("SEM_COARSE_PLANES", planes)
        s = sem.Solver(4, 4, 4, xyz, 1, 3, bc=(1, 1, 1, 1, 0, 0), opts=o)
        b = s.rhs(t.ones(s.levels[0].nlocal, dtype=t.float64, device="cuda"))
        _, info = s.solve(b, rtol=1e-30, maxit=1, allow_noconv=True)
        assert info.coarse_iters == 0
        out.append(s.vcycle(b))
    assert bool(t.isfinite(out[0]).all()) and t.equal(*out)


def test_singular_level_goes_to_the_cg():
    t = __import__("torch")
    o = sem.make_opts(schedule=(3, 1), lambda_override=[2.6], coarse_solver=sem.COARSE_DIRECT)
    s = sem.Solver(4, 4, 4, wl.box_vertices(4, 4, 4), 1, 3, bc=(0,) * 6, opts=o)
    X = s.coords(0)
    b = s.apply_A(t.cos(3.141592653589793 * X[0]))
    _, info = s.solve(b, rtol=1e-30, maxit=1, allow_noconv=True)
    assert info.coarse_iters > 0
