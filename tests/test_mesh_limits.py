"""Meshes with more elements than the 32-bit counts take are refused by pc_create
before anything is built from them: no device call is made, so the refusal is
the same without a GPU."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("nt,message", [(59_652_324, b"59,652,323 triangles"), (238_700_000, b"59,652,323 triangles"),
                                        (1 << 28, b"2^28 triangles")])
def test_too_many_triangles_are_refused_at_once(nt, message):
    from paper_2008_00409_amd import binding
    L = binding.lib()
    tris = np.zeros(3 * nt, dtype=np.int32)     # read once, never written: the kernel's zero page
    rest, mass = np.zeros((3, 3)), np.ones(3)
    m = binding.PcMesh()
    m.nv, m.nt = 3, nt
    m.tris = tris.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))
    m.rest = rest.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    m.mass = mass.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    params = binding.make_params(0.01)
    h = ctypes.c_void_p()
    assert L.pc_create(ctypes.byref(m), ctypes.byref(params), ctypes.byref(h)) == binding.PC_ERR_ARG
    assert message in L.pc_last_error(None) and not h
