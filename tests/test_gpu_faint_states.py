"""States of densities whose reciprocal overflows: the step and the fluid
kernels are linear in the density at constant tau, so such a state steps like
the same state times a power of two, to the spacing of subnormal numbers."""
import numpy as np
import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import balanced

pytestmark = pytest.mark.gpu

SCALE, SPACING = 2.0 ** -1026, 2.0 ** -1074


def _solver(f, nv, f0, hybrid=False):
    s = D.Solver(D.Mesh(f), D.make_params(nv, 4.5, precision=D.PREC_FP64, tau_mode=I.TAU_CONST, tau_or_kn=0.05,
                                          hybrid=hybrid))
    s.set_f_canonical(f0)
    return s


def _start(f, nv):
    """smooth Maxwellians in multiples of 2^-48, so that the scaled state is exact"""
    s = D.Solver(D.Mesh(f), D.make_params(nv, 4.5, precision=D.PREC_FP64, tau_mode=I.TAU_CONST, tau_or_kn=0.05))
    s.init_maxwellian(I.fields("sines", I.leaf_centres(f)[D.Mesh(f).tables()["input"]], seed=4))
    return np.round(s.f_canonical().cpu().numpy() * 2.0 ** 48) * 2.0 ** -48


# the roundings of a step are below SPACING each; through the moments they reach
# a value at most (2 vmax)^3 times the Maxwellian of unit density, and the
# temperature's by as much again times |xi|^2 / 2
TOL = 1024 * SPACING


@pytest.mark.parametrize("nv", [4, 8, 12, 16, 24])
@pytest.mark.parametrize("mesh", ["uniform", "jumps"])
def test_step_of_a_faint_state_is_the_scaled_step(nv, mesh):
    f = I.uniform_forest((3, 2, 2), 0) if mesh == "uniform" else balanced(I.random_forest(5, (2, 2, 2), 2, 0.3))
    f0 = _start(f, nv)
    a, b = _solver(f, nv, f0), _solver(f, nv, f0 * SCALE)
    for s in (a, b):
        s.step(2, cfl=0.5)
        assert s.check()[0] == D.OK
    fa, fb = a.f_canonical().cpu().numpy(), b.f_canonical().cpu().numpy()
    assert np.abs(fb).max() > 2.0 ** 30 * TOL
    assert np.abs(fb - fa * SCALE).max() <= TOL


def test_fluid_cells_of_a_faint_state_step_like_the_scaled_state():
    f, nv = I.uniform_forest((3, 2, 2), 0), 8
    f0 = _start(f, nv)
    a, b = _solver(f, nv, f0, True), _solver(f, nv, f0 * SCALE, True)
    mask = np.zeros(a.n, np.uint8)
    mask[:4] = 1
    for s in (a, b):
        s.hybrid_step(mask, n=2, cfl=0.5)
        assert s.check()[0] == D.OK
    ma, mb = a.mom.cpu().numpy(), b.mom.cpu().numpy()
    # six fluxes of three sums over half an axis each, of terms up to |xi|^3
    assert np.abs(mb).max() > 2.0 ** 28 * TOL
    assert np.abs(mb - ma * SCALE).max() <= 64 * TOL
