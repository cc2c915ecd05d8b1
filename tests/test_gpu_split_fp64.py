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


@pytest.mark.parametrize("mesh", ["walls", "jumps", "uniform"])
def test_the_pair_is_one_launch_of_576_threads_bitwise(mesh):
    """the default, whatever dvm_tune_split says, (576, 30) and a batch: one step"""
    f = {"walls": _forest(), "jumps": balanced(I.random_forest(5, (2, 3, 2), 2, 0.3)),
         "uniform": I.uniform_forest((3, 3, 3), 0)}[mesh]
    f1, m1 = _stepped(f, (576, 30), steps=3)
    for shape, split, irr in ((None, None, (0, 0)), (None, 0, (0, 0)), (None, 1, (0, 0)), (None, 1, (576, 71)),
                              ((192, 21), None, (0, 0))):
        f2, m2 = _stepped(f, shape, split, irr, steps=3)
        assert np.array_equal(f1, f2) and np.array_equal(m1, m2), (shape, split, irr)
    b = _solver(f, 24, D.PREC_FP64)
    D.Batch([b], cfl=0.5).step(3)
    assert np.array_equal(f1, b.f_canonical().cpu().numpy()) and np.array_equal(m1, b.mom.cpu().numpy())


def test_a_second_launch_of_its_own_steps_the_other_cells_of_the_pair():
    """dvm_tune_split(1, 192, 31) with the pair's shape: its regular cells as
    ever, the others by 192 threads"""
    f = _forest()
    reg = _regular(f)
    pair, narrow = _stepped(f, None), _stepped(f, (192, 31))
    both = _stepped(f, None, 1, (192, 31))
    assert np.array_equal(both[0][reg], pair[0][reg]) and np.array_equal(both[1][:, reg], pair[1][:, reg])
    assert np.array_equal(both[0][~reg], narrow[0][~reg]) and np.array_equal(both[1][:, ~reg], narrow[1][:, ~reg])


def test_without_regular_cells_the_pair_is_not_tuned():
    """one cell between walls: its only launch is (576, 51), listed by itself"""
    s = _solver(I.uniform_forest((1, 1, 1), 0, bc=(I.WALL,) * 6), 24, D.PREC_FP64)
    for _ in range(3):
        s.tune(reps=1)
        assert s.get_shape()[:2] in s.shapes() and s.get_shape()[:2] != (192, 21)
    t = _solver(I.uniform_forest((1, 1, 1), 0, bc=(I.WALL,) * 6), 24, D.PREC_FP64)
    u = _solver(I.uniform_forest((1, 1, 1), 0, bc=(I.WALL,) * 6), 24, D.PREC_FP64)
    u.set_shape(576, 30, 1, 0)
    for x in (t, u):
        x.step(2, cfl=0.5)
    assert np.array_equal(t.f_canonical().cpu().numpy(), u.f_canonical().cpu().numpy())


@pytest.mark.parametrize("shape,frac", [((16, 4, 4), 0.0), ((257, 1, 1), 0.0), ((8, 8, 8), 0.2857), ((8, 8, 8), 0.2877)],
                         ids=str)
def test_the_default_on_both_sides_of_the_pairs_smallest_mesh(shape, frac):
    """256 and 257 cells, all regular; 1,534 and 1,541 with level jumps"""
    f = I.uniform_forest(shape, 0)
    if frac:
        mask = np.zeros(len(f.level), bool)
        mask[np.random.default_rng(3).permutation(len(f.level))[:round(frac * len(f.level))]] = True
        f = I.refine(f, mask)
    f1, m1 = _stepped(f, (576, 30), steps=2)
    f2, m2 = _stepped(f, None, steps=2)
    assert np.array_equal(f1, f2) and np.array_equal(m1, m2)


def test_the_default_on_a_small_mesh_is_as_fast_as_one_launch():
    """27 cells between walls: two launches take 1.8 times the one's time"""
    import time
    import torch
    f = I.uniform_forest((3, 3, 3), 0, 1.0 / 3, WALLS)
    a, b = _solver(f, 24, D.PREC_FP64), _solver(f, 24, D.PREC_FP64)
    b.set_shape(576, 30, *b.get_shape()[2:])
    best = [np.inf, np.inf]
    for _ in range(20):
        for k, s in enumerate((a, b)):
            torch.cuda.synchronize()
            t = time.perf_counter()
            s.step(100, cfl=0.5)
            torch.cuda.synchronize()
            best[k] = min(best[k], time.perf_counter() - t)
    assert best[0] <= 1.25 * best[1]
