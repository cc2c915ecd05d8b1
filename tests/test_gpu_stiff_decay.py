"""A stiff collision (dt many times tau) where f is far above its Maxwellian:
what is left there is exp(-dt / tau) f, to the last digits of the storage
precision, however small the factor is."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv", [8, 12, 24])
@pytest.mark.parametrize("x", [1.0, 10.0, 20.0, 30.0, 40.0])
@pytest.mark.parametrize("precision", [D.PREC_FP64, D.PREC_FP32])
def test_tail_of_a_cold_cell_decays_like_the_exponential(nv, x, precision):
    """one periodic cell (its transport cancels exactly): a cold Maxwellian and
    a faint beam in the eight corners of velocity space, where the Maxwellian is
    far below what the decay leaves of the beam"""
    f = I.uniform_forest((1, 1, 1), 0)
    om = O.Mesh(f)
    tau = 0.0625
    o = O.Solver(om, O.make_params((nv,) * 3, (-4.5,) * 3, (4.5,) * 3, tau_or_kn=tau))
    o.init_maxwellian(np.array([[1.0], [0.0], [0.0], [0.0], [0.3]]))
    f0 = o.get_f().copy().reshape(nv, nv, nv)
    f0[::nv - 1, ::nv - 1, ::nv - 1] = 1e-4
    if precision == D.PREC_FP32:
        f0 = f0.astype(np.float32).astype(np.float64)
    o.set_f(f0.reshape(1, -1))
    assert o.step(x * tau, 1) == 0
    s = D.Solver(D.Mesh(f), D.make_params(nv, 4.5, precision=precision, tau_mode=I.TAU_CONST, tau_or_kn=tau))
    s.set_f_canonical(f0.reshape(1, -1))
    s.step(1, dt=x * tau)
    assert s.check()[0] == D.OK
    ref = o.get_f().reshape(nv, nv, nv)[::nv - 1, ::nv - 1, ::nv - 1]
    got = s.f_canonical().double().cpu().numpy().reshape(nv, nv, nv)[::nv - 1, ::nv - 1, ::nv - 1]
    assert np.abs(ref / (np.exp(-x) * f0[0, 0, 0]) - 1).max() < 1e-9  # the beam's decay, next to nothing else
    # x to an ulp on both sides, the exponential and the products to a few
    tol = (2 * x + 8) * 2.0 ** -53 if precision == D.PREC_FP64 else (2 * x + 8) * 2.0 ** -53 + 2 * 2.0 ** -24
    assert np.abs(got / ref - 1).max() <= tol
