"""The Korobov kernel on every tile it picks (4, 8 and 16 cells, a last tile
that is partly empty) and both ways it sums the collision frequency (the
matrix product, the partner lists of few trials), against the FP64 oracle."""
import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I
from tests.gpu_common import Case
from tests.test_gpu_parity import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv,base,p", [(8, (3, 3, 1), 131), (8, (13, 11, 11), 31), (8, (13, 11, 11), 131),
                                       (8, (16, 16, 13), 131), (8, (16, 16, 13), 31), (4, (3, 1, 1), 31),
                                       (4, (5, 3, 3), 127), (4, (17, 16, 16), 61), (12, (3, 2, 1), 61)])
@pytest.mark.parametrize("prec,tol", [(D.PREC_FP32, 2e-5), (D.PREC_FP64, 1e-12)])
def test_korobov_tiles(nv, base, p, prec, tol):
    f = I.uniform_forest(base, 0, 1.0 / base[0])
    case = Case(f, nv, 3.0 if nv == 4 else 4.5, collision=I.COLL_KOROBOV, tau=0.5, korobov_p=p, fields="sines",
                field_args={"seed": 3})
    _compare(case, 1, prec, tol, f_tol=tol)
