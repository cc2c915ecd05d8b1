"""The LBM kernel's list of FINER faces where it can go wrong (a workgroup of
256 cells with more FINER faces than the list holds, one with none, a last
wave that is partly empty), against the FP64 oracle, and the layout conversion
at the edges of its tiles."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import balanced

pytestmark = pytest.mark.gpu


def _islands():
    """32 x 16 x 16 roots, all refined but the last 128 of the first 16^3 block
    in Morton order and the first 128 of the second: cells 31744 .. 31999, one
    workgroup, have 320 FINER faces."""
    f = I.uniform_forest((32, 16, 16), 0, 1.0 / 32)
    x, y, z = f.ijk.T
    coarse = ((x >= 8) & (x < 16) & (y >= 12) & (z >= 12)) | ((x >= 16) & (x < 24) & (y < 4) & (z < 4))
    return I.refine(f, ~coarse)


def _run(forest, q, prec, steps=3):
    om = O.Mesh(forest)
    t = om.tables()
    x = I.leaf_centres(forest)[t["input"]]
    prim = np.stack([1 + 0.1 * np.sin(2 * np.pi * x[:, 0]), 0.06 * np.cos(2 * np.pi * x[:, 1]),
                     0.05 * np.sin(2 * np.pi * x[:, 2]), 0.04 * np.cos(2 * np.pi * x[:, 0])])
    o = O.Solver(om, O.lbm_params(q, 0.6))
    o.init_lbm(prim)
    s = D.LBM(D.Mesh(forest), q=q, precision=prec, tau=0.6)
    s.init(prim)
    dt = s.dt(0.5)
    assert o.step(dt, steps) == 0
    s.step(steps, dt=dt)
    return t, o.get_f(), s.f_canonical().double().cpu().numpy()


@pytest.mark.parametrize("q,prec,tol", [(19, D.PREC_FP32, 2e-5), (27, D.PREC_FP32, 2e-5), (19, D.PREC_FP64, 1e-12),
                                        (27, D.PREC_FP64, 1e-12)])
def test_lbm_more_finer_faces_than_the_list_holds(q, prec, tol):
    t, fo, fg = _run(_islands(), q, prec)
    finer = (np.asarray(t["type"]) == 2).sum(1)
    assert finer[31744:32000].sum() == 320
    assert np.abs(fg - fo).max() <= tol * np.abs(fo).max()


@pytest.mark.parametrize("base,level", [((1, 1, 1), 0), ((3, 7, 3), 0), ((13, 5, 1), 0), ((5, 13, 17), 0)])
def test_lbm_ragged_uniform(base, level):
    _, fo, fg = _run(I.uniform_forest(base, level, 1.0 / base[0]), 19, D.PREC_FP64)
    assert np.abs(fg - fo).max() <= 1e-12 * np.abs(fo).max()


@pytest.mark.parametrize("n", [1, 127, 128, 129, 257])
@pytest.mark.parametrize("q", [19, 27])
def test_lbm_layout_round_trip(n, q):
    s = D.LBM(D.Mesh(I.uniform_forest((n, 1, 1), 0, 1.0)), q=q, precision=D.PREC_FP64)
    f = np.random.default_rng(n).random((n, 27))
    if q == 19:
        for k in range(27):
            if abs(k // 9 - 1) + abs(k // 3 % 3 - 1) + abs(k % 3 - 1) == 3:
                f[:, k] = 0.0
    s.set_f_canonical(f)
    assert np.array_equal(s.f_canonical().cpu().numpy(), f)
