"""The x-faces summed inside workgroups of 4 and of 8 elements along x, and the steps the
FDM takes as it reads A's output, with the direction passes after them (SEM_GS_ALL=0:
levels of a few elements take one launch instead by default): the FP32 RAS local
solves with FP32, FP16 and BF16 operands against the oracle (SEM_XGROUP=8 is taken up
to p = 7), the product at p = 7 against the form that leaves every x-face to the passes
(the same sums in the same order, bit for bit), and several right sides in one launch."""
import numpy as np
import pytest

from pairs import Pair, dev, host, rel_err
from paper_2110_07663_amd import sem
from paper_2110_07663_amd import workloads as wl

pytestmark = pytest.mark.gpu

GROUPS = [(2, (8, 2, 1), (1,) * 6, "8"), (3, (8, 2, 2), (0, 1, 0, 1, 1, 0), "8"),
          (3, (4, 3, 1), (1, 0, 1, 1, 0, 1), "4"), (5, (16, 1, 2), (1, 0, 0, 1, 1, 1), "8"),
          (5, (12, 1, 1), (1,) * 6, "4"), (7, (8, 2, 2), (0, 1, 1, 0, 1, 1), "8"),
          (7, (4, 3, 2), (1, 0, 1, 1, 0, 1), "4"), (7, (12, 1, 2), (1, 1, 0, 0, 1, 0), "4"),
          (8, (8, 2, 1), (0, 0, 1, 1, 0, 1), "8"), (9, (4, 2, 2), (0, 1, 1, 1, 0, 0), "4")]


@pytest.mark.parametrize("p,shape,bc,group", GROUPS)
def test_ras_sums_x_faces(monkeypatch, p, shape, bc, group):
    t = __import__("torch")
    monkeypatch.setenv("SEM_GS_ALL", "0")
    monkeypatch.setenv("SEM_XGROUP", group)
    want = None
    for fdm, tol, xstep, ystep in (
            (sem.F32, 1e-5, "1", "1"), (sem.F32, 1e-5, "1", "0"), (sem.F32, 1e-5, "0", "1"),
            (sem.F16, 5e-3, "1", "1"), (sem.F16, 5e-3, "0", "1"), (sem.BF16, 4e-2, "1", "1")):
        monkeypatch.setenv("SEM_FDM_XSTEP", xstep)
        monkeypatch.setenv("SEM_FDM_YSTEP", ystep)
        P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother="ras", bc=bc, cheb_order=2,
                 smoother_prec=sem.F32, fdm_prec=fdm, lambda_override=[1.8], oracle=want is None)
        r, ro = P.random_local(41)
        b, bo = P.random_local(42)
        if want is None:
            want = P.ora.levels[0].apply_S(ro), P.ora.smooth(bo, ro, level=0)
        x = r.to(t.float32)
        tag = (fdm, xstep, ystep)
        assert rel_err(host(P.gpu.apply_S(x)), want[0]) < tol, tag
        assert rel_err(host(P.gpu.smooth(b.to(t.float32), x)), want[1]) < tol, tag


@pytest.mark.parametrize("p,shape,bc,group", [g for g in GROUPS if g[0] == 7])
def test_ax_sums_x_faces(monkeypatch, p, shape, bc, group):
    t = __import__("torch")
    monkeypatch.setenv("SEM_GS_ALL", "0")
    monkeypatch.setenv("SEM_XGROUP", group)
    for prec, geom in ((t.float64, sem.F32), (t.float32, sem.F32), (t.float32, sem.F16)):
        out = []
        for fuse in ("0", "1"):
            monkeypatch.setenv("SEM_AX_XFUSE", fuse)
            P = Pair(shape, p, mesh="sin", schedule=(p, 1), smoother_prec=sem.F32, geom_prec=geom,
                     bc=bc, lambda_override=[2.0], oracle=False)
            out.append(host(P.gpu.apply_A(P.random_local(43)[0].to(prec))))
        np.testing.assert_array_equal(*out)


@pytest.mark.parametrize("shape,group,fdm,geom", [((8, 2, 2), "8", sem.F32, sem.F32),
                                                  ((4, 2, 2), "4", sem.F16, sem.F16)])
def test_several_right_sides(monkeypatch, shape, group, fdm, geom):
    t = __import__("torch")
    monkeypatch.setenv("SEM_GS_ALL", "0")
    monkeypatch.setenv("SEM_XGROUP", group)
    opts = sem.make_opts(schedule=(7, 3, 1), smoother=sem.SMOOTH_RAS, smoother_prec=sem.F32,
                         batch_rhs=3, fdm_prec=fdm, geom_prec=geom)
    S = sem.Solver(*shape, wl.sampled_mesh(*shape, sem.gll_nodes(7)[0], wl.sin_map(0.05)), 7, 7,
                   opts=opts)
    X = host(S.coords(0))
    bs = [S.rhs(dev(wl.sinusoid(1 + k, 1, 2)[0](X[0], X[1], X[2]))) for k in range(3)]
    out = {}
    for mode in ("1", "0"):
        monkeypatch.setenv("SEM_BATCH_JOINT", mode)
        xs = [t.zeros_like(b) for b in bs]
        infos = sem.batch_solve([S], [bs], [xs], rtol=1e-8, maxit=100)
        assert all(i.converged and i.true_rel_res <= 1e-8 for i in infos)
        out[mode] = [host(x) for x in xs]
    for a, b in zip(out["1"], out["0"]):
        np.testing.assert_array_equal(a, b)
