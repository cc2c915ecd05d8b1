"""The MUSCL step where level jumps lie between cells that touch walls: those have
no slope, so the cells beyond them must not count.  Meshes one cell deep, of walled
cells alone or of a few without a wall between them, against the FP64 oracle."""
import numpy as np
import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import Case
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu

BCS = (I.INFLOW, I.OUTFLOW, I.WALL, I.WALL, I.PERIODIC, I.PERIODIC)


@pytest.mark.parametrize("nv", [8, 12, 24])
@pytest.mark.parametrize("prec,tol", [(D.PREC_FP32, 2e-5), (D.PREC_FP64, 1e-12)])
@pytest.mark.parametrize("n,refined", [((2, 1, 2), (0,)), ((2, 1, 3), (1, 2, 4)), ((3, 2, 3), (0, 4, 11))],
                         ids=["one", "three", "between"])
def test_muscl_jumps_between_walls(nv, prec, tol, n, refined):
    f = I.uniform_forest(n, 0, 1.0 / n[0], BCS)
    mask = np.zeros(len(f.level), bool)
    mask[list(refined)] = True
    f = I.refine(f, mask)
    case = Case(f, nv, 6.0, scheme=I.SCHEME_MUSCL, tau=0.05, fields="sines",
                field_args={"seed": 3}, inflow=(1.0, 0.4, 0.0, 0.0, 1.0), t_wall=1.1)
    _compare(case, 3, prec, tol, f_tol=tol)
