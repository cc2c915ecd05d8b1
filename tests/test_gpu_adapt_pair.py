"""FP64 at 24^3 nodes on a mesh adapted on the device: the default pair of
launches steps from the selection list that the adaptation built."""
import numpy as np
import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import Case, balanced, moment_errors, oracle_run
from tests.test_gpu_adapt import _flags, _sorted_forest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [0, 2])
def test_adapted_fp64_24_default_step(seed):
    import torch
    bcs = (I.PERIODIC,) * 6 if seed == 0 else (I.INFLOW, I.OUTFLOW, I.WALL, I.OUTFLOW, I.PERIODIC, I.PERIODIC)
    f0 = _sorted_forest(balanced(I.random_forest(seed, (2, 2, 2), 3, 0.25, bcs)))
    fl = _flags(f0, np.random.default_rng(60 + seed))
    make = lambda m: D.Solver(m, D.make_params(24, 6.0, precision=D.PREC_FP64, tau_or_kn=0.1))
    keep = D.Mesh(f0)
    s = make(keep)
    f1, m1, a = D.adapt(s, fl)
    m2 = D.Mesh(f1)
    b, c = make(m2), make(m2)
    c.set_shape(576, 30, 1, 0)
    prim = I.fields("sines", I.leaf_centres(f1), seed=seed)
    for x in (a, b, c):
        x.init_maxwellian(prim)
        x.step(3, cfl=0.5)
        assert x.check()[0] == D.OK
    assert a.get_shape()[:2] == b.get_shape()[:2] == (192, 21)
    torch.cuda.synchronize()
    for x in (b, c):
        assert torch.equal(a.f_canonical(), x.f_canonical())
        assert torch.equal(a.mom, x.mom)
    case = Case(f1, 24, 6.0, tau=0.1, fields="sines", field_args={"seed": seed})
    o = oracle_run(case, 3)
    assert np.all(moment_errors(a.mom.cpu().numpy(), o["mom"]) <= 1e-12)


@pytest.mark.parametrize("seed", [0, 2])
def test_adapted_fp64_24_split_step(seed):
    """the same few cells, two launches over the device's list asked for"""
    bcs = (I.PERIODIC,) * 6 if seed == 0 else (I.INFLOW, I.OUTFLOW, I.WALL, I.OUTFLOW, I.PERIODIC, I.PERIODIC)
    f0 = _sorted_forest(balanced(I.random_forest(seed, (2, 2, 2), 3, 0.25, bcs)))
    fl = _flags(f0, np.random.default_rng(60 + seed))
    keep = D.Mesh(f0)
    s = D.Solver(keep, D.make_params(24, 6.0, precision=D.PREC_FP64, tau_or_kn=0.1))
    f1, m1, a = D.adapt(s, fl)
    m2 = D.Mesh(f1)
    b = D.Solver(m2, D.make_params(24, 6.0, precision=D.PREC_FP64, tau_or_kn=0.1))
    prim = I.fields("sines", I.leaf_centres(f1), seed=seed)
    a.split(1)
    b.set_shape(576, 30, 1, 0)
    for x in (a, b):
        x.init_maxwellian(prim)
        x.step(3, cfl=0.5)
        assert x.check()[0] == D.OK
    assert np.array_equal(a.f_canonical().cpu().numpy(), b.f_canonical().cpu().numpy())
    assert np.array_equal(a.mom.cpu().numpy(), b.mom.cpu().numpy())
