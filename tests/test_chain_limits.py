"""The chain bodies' index limits, checked on the library's own host functions
(CPU only, no device calls)."""
import ctypes as C

import numpy as np
import pytest


@pytest.fixture(scope="module")
def P():
    import os
    import paper_1411_4622_amd as P
    if not os.path.exists(P.LIB_PATH):
        from paper_1411_4622_amd import build
        build.build()
    P.load()
    return P


@pytest.mark.parametrize("dtype,most", [("f64", 1 << 29), ("f32", 1 << 30), ("u8", 1 << 30)])
def test_register_bodies_take_what_32_bit_offsets_reach(P, dtype, most):
    """pila::piped_allowed: the pipelined and long-row bodies form byte offsets
    into the lengths and into the four-byte ray indices in 32 bits, so the
    wider of the two bounds the entries (1300 x 1300, 720 angles and one-byte
    lengths are 1.2e9)."""
    from paper_1411_4622_amd._binding import CCsr
    allowed = P.load()._ZN4pila13piped_allowedEPK9pila_geomPK8pila_csr
    allowed.restype = C.c_bool
    geom = P.Geometry(1300, np.zeros(720), 1839, None, dtype)
    csr = CCsr()
    csr.max_row = 1440
    for nnz, want in ((1, True), (most, True), (most + 1, False), (1 << 32, False), (0, False)):
        csr.nnz = nnz
        assert allowed(C.byref(geom.c), C.byref(csr)) is want, nnz
