"""The MUSCL step of cells with level jumps in their stencil, on every velocity
grid the library has (one to three slots a thread, FP32 through LDS and FP64
through registers), against the FP64 oracle: three levels, so that finer cells
lie behind finer and coarser ones, and inflow, outflow and wall faces."""
import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import Case, balanced
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu

BCS = (I.INFLOW, I.OUTFLOW, I.WALL, I.WALL, I.PERIODIC, I.PERIODIC)


@pytest.mark.parametrize("nv", [4, 12, 16, 24])
@pytest.mark.parametrize("prec,tol", [(D.PREC_FP32, 2e-5), (D.PREC_FP64, 1e-12)])
@pytest.mark.parametrize("bcs", [(I.PERIODIC,) * 6, BCS], ids=["periodic", "walls"])
def test_muscl_three_levels(nv, prec, tol, bcs):
    f = balanced(I.random_forest(11, (3, 3, 2), 2, 0.12, bcs))
    assert f.level.max() == 2
    case = Case(f, nv, 3.0 if nv == 4 else 6.0, scheme=I.SCHEME_MUSCL, tau=0.05, fields="sines",
                field_args={"seed": 5}, inflow=(1.0, 0.3, 0.0, 0.0, 1.0), t_wall=1.1)
    _compare(case, 3, prec, tol, f_tol=tol)
