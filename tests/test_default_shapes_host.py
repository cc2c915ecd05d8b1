"""The default kinds of stores by size (host only: no device call)."""
import ctypes as C

import pytest

from paper_1503_00707_amd import dvm as D
from paper_1503_00707_amd import inputs as I


@pytest.mark.parametrize("precision,nv,shape,nt", [
    # FP32, 12^3 and 24^3 nodes: non-temporal below 24 MiB and above 128 MiB a buffer; 16^3: always
    (D.PREC_FP32, 24, (3, 4, 5), 1), (D.PREC_FP32, 24, (5, 7, 13), 1), (D.PREC_FP32, 24, (3, 8, 19), 0),
    (D.PREC_FP32, 24, (11, 13, 16), 0), (D.PREC_FP32, 24, (11, 13, 17), 1), (D.PREC_FP32, 16, (7, 8, 9), 1),
    (D.PREC_FP32, 16, (11, 12, 13), 1), (D.PREC_FP32, 12, (9, 10, 11), 1), (D.PREC_FP32, 12, (16, 17, 18), 0), (D.PREC_FP32, 8, (7, 8, 9), 0),
    # FP64: above 128 MiB, 24^3 nodes above 40
    (D.PREC_FP64, 24, (3, 4, 5), 0), (D.PREC_FP64, 16, (7, 8, 9), 0), (D.PREC_FP64, 16, (16, 16, 17), 1),
    (D.PREC_FP64, 24, (6, 7, 8), 0), (D.PREC_FP64, 24, (7, 8, 9), 1), (D.PREC_FP64, 24, (12, 12, 12), 1)], ids=str)
def test_kind_of_stores_by_size(precision, nv, shape, nt):
    m = D.Mesh(I.uniform_forest(shape, 0))
    h = C.c_void_p()
    p = D.make_params(nv, 6.0, precision=precision)
    assert D.lib().dvm_create_solver(m.h, C.byref(p), C.byref(h)) == D.OK
    v = [C.c_int32() for _ in range(4)]
    assert D.lib().dvm_tune_get(h, *(C.byref(x) for x in v)) == D.OK
    D.lib().dvm_destroy_solver(h)
    assert v[3].value == nt
