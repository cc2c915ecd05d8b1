"""dvm_tune_split at 24^3 nodes in FP64.  Workgroups of 192 and of 576 threads
add the terms of a moment in another order, which shows in the last bits, so
that each cell tells which kernel stepped it."""
import numpy as np
import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import balanced
from tests.test_gpu_default_shapes import WALLS, _solver

pytestmark = pytest.mark.gpu


def _forest():
    return balanced(I.random_forest(9, (2, 2, 2), 3, 0.25, WALLS))


def _stepped(f, shape, split=None, irr=(0, 0), steps=1):
    s = _solver(f, 24, D.PREC_FP64)
    if shape:
        s.set_shape(*shape, 32, 1)
    if split is not None:
        s.split(split, *irr)
    s.step(steps, cfl=0.5)
    assert s.check()[0] == D.OK
    return s.f_canonical().cpu().numpy(), s.mom.cpu().numpy()


def _regular(f):
    ty = np.asarray(D.Mesh(f).tables()["type"])
    return ~((ty == 2) | (ty == 5)).any(1)  # FINER, WALL


@pytest.mark.parametrize("irr", [(0, 0), (576, 51)])
def test_split_of_192_threads_steps_the_other_cells_at_576(irr):
    f = _forest()
    reg = _regular(f)
    narrow, wide = _stepped(f, (192, 31)), _stepped(f, (576, 30))
    both = _stepped(f, (192, 31), 1, irr)
    assert reg.any() and not reg.all()
    assert not np.array_equal(narrow[1][:, reg], wide[1][:, reg])
    assert not np.array_equal(narrow[1][:, ~reg], wide[1][:, ~reg])
    assert np.array_equal(both[0][reg], narrow[0][reg]) and np.array_equal(both[1][:, reg], narrow[1][:, reg])
    assert np.array_equal(both[0][~reg], wide[0][~reg]) and np.array_equal(both[1][:, ~reg], wide[1][:, ~reg])
