"""Which transfer kernels a shape runs: the rule of csrc/intergrid_mfma.hip, called
in the built library (host code only)."""

import ctypes as C

import numpy as np
import pytest

from paper_2211_13719_amd._lib import lib


class AggGeom(C.Structure):
    _fields_ = [("L", C.c_int * 4), ("b", C.c_int * 4), ("C", C.c_int * 4), ("V", C.c_int), ("Vc", C.c_int)]


_leads = lib["_ZN4mrhs22intergrid_staged_leadsEbbRKNS_7AggGeomEii"]
_leads.restype, _leads.argtypes = C.c_bool, (C.c_bool, C.c_bool, C.POINTER(AggGeom), C.c_int, C.c_int)


def staged_leads(prec, prolong, dims, block, h, nrhs):
    a = AggGeom()
    for m in range(4):
        a.L[m], a.b[m], a.C[m] = dims[m], block[m], dims[m] // block[m]
    a.V, a.Vc = int(np.prod(dims)), int(np.prod(dims)) // int(np.prod(block))
    return _leads(prec == "bf16", prolong, C.byref(a), h, nrhs)


@pytest.mark.parametrize("prec,prolong,dims,block,h,nrhs", [
    # us of the other kernel, staged
    ("f32", False, (4, 4, 4, 4), (4, 4, 4, 4), 6, 64),       # 32.8, 41.5
    ("f32", False, (8, 8, 8, 4), (4, 4, 4, 4), 6, 48),       # 32.5, 41.1
    ("f32", False, (8, 8, 8, 4), (4, 4, 4, 2), 6, 33),       # 18.5, 22.6
    ("f32", False, (16, 16, 4, 4), (4, 4, 2, 2), 6, 48),     # 13.4, 14.2
    ("f32", False, (4, 4, 4, 8), (2, 2, 2, 2), 16, 48),      # 8.2, 10.5
    ("f32", False, (8, 4, 4, 4), (4, 4, 4, 4), 16, 64),      # 73, 105
    ("bf16", False, (12, 12, 8, 8), (4, 4, 4, 4), 6, 64),    # 16.3, 22.8
    ("bf16", False, (16, 16, 8, 8), (4, 4, 4, 4), 6, 48),    # 19.2, 24.1
    ("bf16", False, (8, 8, 4, 4), (2, 2, 2, 2), 16, 48),     # 5.8, 6.7
    ("bf16", False, (8, 8, 8, 8), (4, 4, 4, 4), 6, 24),      # 13.6, 13.5
    ("bf16", False, (16, 16, 8, 4), (4, 4, 2, 2), 6, 48),    # 9.8, 11.4
    ("f32", True, (8, 8, 4, 4), (2, 2, 2, 2), 6, 48),        # 6.3, 8.0
    ("bf16", True, (16, 16, 6, 6), (4, 4, 2, 2), 6, 48),     # 13.6, 16.3
])
def test_other_kernels_where_they_lead(prec, prolong, dims, block, h, nrhs):
    assert not staged_leads(prec, prolong, dims, block, h, nrhs)


@pytest.mark.parametrize("prec,prolong,dims,block,h,nrhs", [
    ("f32", False, (24, 24, 24, 24), (4, 4, 4, 4), 6, 24),   # 400, 245
    ("f32", False, (4, 4, 4, 4), (4, 4, 4, 4), 6, 32),       # 32.2, 25.4
    ("f32", False, (12, 12, 12, 12), (4, 4, 4, 4), 6, 64),   # 59.9, 44.9
    ("f32", False, (16, 16, 16, 16), (2, 2, 2, 2), 16, 48),  # 22.6, 18.7
    ("bf16", False, (12, 12, 12, 12), (4, 4, 4, 4), 6, 33),  # 33.8, 23.1
    ("f32", False, (16, 8, 8, 4), (4, 2, 2, 2), 6, 40),      # 0.88 of the other
    ("bf16", False, (4, 4, 4, 4), (4, 4, 4, 4), 6, 16),      # 13.2, 10.9
    ("f32", True, (4, 4, 4, 4), (4, 4, 4, 4), 6, 64),        # 37.9, 8.8
    ("bf16", True, (16, 16, 16, 16), (4, 4, 4, 4), 6, 48),   # 0.86
])
def test_staged_kernels_where_they_lead(prec, prolong, dims, block, h, nrhs):
    assert staged_leads(prec, prolong, dims, block, h, nrhs)
