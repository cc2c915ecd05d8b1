"""The default shapes of the step: runs of cells per XCD and kinds of stores
chosen by size, and the two launches of FP64 at 24^3 nodes, against one launch
over all cells in input order: the same step, bitwise where the workgroups are
the same."""
import numpy as np
import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import balanced

pytestmark = pytest.mark.gpu

WALLS = (I.INFLOW, I.OUTFLOW, I.WALL, I.OUTFLOW, I.PERIODIC, I.PERIODIC)


def _solver(f, nv, precision):
    dm = D.Mesh(f)
    s = D.Solver(dm, D.make_params(nv, 4.5, precision=precision, tau_mode=I.TAU_CONST, tau_or_kn=0.05,
                                   inflow=(1.0, 0.5, 0.0, 0.0, 1.0), t_wall=1.1))
    s.init_maxwellian(I.fields("sines", I.leaf_centres(f)[dm.tables()["input"]], seed=31))
    return s


# one cell; fewer than a run; all regular; level jumps; level jumps and walls; the last sizes cross 128 MiB of FP64 state
@pytest.mark.parametrize("shape,nv", [((1, 1, 1), 24), ((1, 1, 7), 24), ((5, 5, 5), 24), ("jumps", 24), ("walls", 24),
                                      ("walls", 16), ("walls", 12), ("walls", 8), ((16, 16, 16), 16),
                                      ((16, 16, 17), 16)], ids=str)
@pytest.mark.parametrize("precision", [D.PREC_FP64, D.PREC_FP32])
def test_default_shape_is_one_plain_launch_bitwise(shape, nv, precision):
    if shape == "jumps":
        f = balanced(I.random_forest(5, (2, 3, 2), 2, 0.3))
    elif shape == "walls":
        f = balanced(I.random_forest(9, (2, 2, 2), 3, 0.25, WALLS))
    else:
        f = I.uniform_forest(shape, 0)
    a, b = _solver(f, nv, precision), _solver(f, nv, precision)
    b.set_shape(*b.get_shape()[:2], 1, 0)
    b.split(0)
    for s in (a, b):
        s.step(3, cfl=0.5)
    assert a.check()[0] == D.OK
    fa, fb = a.f_canonical().cpu().numpy(), b.f_canonical().cpu().numpy()
    ma, mb = a.mom.cpu().numpy(), b.mom.cpu().numpy()
    if precision == D.PREC_FP64 and nv == 24:
        # other workgroups add the 24^3 terms of a moment in another order
        assert np.abs(fa - fb).max() <= 1e-12 * np.abs(fb).max()
        assert np.abs(ma - mb).max() <= 1e-12 * np.abs(mb).max()
    else:
        assert np.array_equal(fa, fb)
        assert np.array_equal(ma, mb)


def test_batch_of_fp64_24_is_the_one_launch_shape_bitwise():
    """a batch has no pair of launches: its default shape there, set on a
    solver, gives the batch's step bitwise; the pair is listed and set too"""
    f = balanced(I.random_forest(9, (2, 2, 2), 3, 0.25, WALLS))
    a, b = _solver(f, 24, D.PREC_FP64), _solver(f, 24, D.PREC_FP64)
    assert b.get_shape()[:2] == (192, 21) and (192, 21) in b.shapes()
    D.Batch([a], cfl=0.5).step(3)
    b.set_shape(576, 30, 32, 1)
    b.step(3, cfl=0.5)
    b.set_shape(192, 21, 32, 1)
    assert np.array_equal(a.f_canonical().cpu().numpy(), b.f_canonical().cpu().numpy())
    assert np.array_equal(a.mom.cpu().numpy(), b.mom.cpu().numpy())
    c = _solver(f, 24, D.PREC_FP32)
    with pytest.raises(RuntimeError):
        c.set_shape(192, 21, 32, 1)
