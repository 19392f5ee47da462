"""Byte model of the amplitude leg of bench.py: the passes it counts are those that the object runs
(pfc_apfc_x_fused), which depends on the row length, the number of fields and the dtype (no GPU)."""
import ctypes
import math
import os
import sys

import pytest

import pfc_inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def _x_fused(shape, kvec, dtype):
    import paper_2603_26818_amd as pfc
    from paper_2603_26818_amd import _binding as b

    lib = pfc.load_library()
    d = b.ApfcDesc()
    d.ndim, d.dtype, d.nfields = len(shape), dtype, len(kvec)
    for a in range(3):
        d.n[a], d.dx[a] = (shape[a], math.pi / 2) if a < len(shape) else (1, 1.0)
    for j, row in enumerate(kvec):
        for a, c in enumerate(row):
            d.k[j][a] = c
    d.dB, d.Bx, d.t, d.v, d.dt = -0.15, 1.0, 0.3, 1.0, 0.5
    h = ctypes.c_void_p()
    assert lib.pfc_apfc_create(ctypes.byref(h), ctypes.byref(d)) == 0
    try:
        return bool(lib.pfc_apfc_x_fused(h))
    finally:
        lib.pfc_apfc_destroy(h)


# rows of a power of two from 16 to 1024; 64 threads per field, at most 512; 512 values (1024 for the longest
# rows) and their padding per field in at most 64 KB of LDS: 4.25 KB in FP32, twice that in FP64
@pytest.mark.parametrize("shape,lattice,dtype,fused", [
    ((256, 256, 256), "bcc", 0, True), ((256, 256, 256), "bcc", 1, True), ((16, 16, 1024), "bcc", 0, True),
    ((16, 16, 1024), "bcc", 1, False), ((64, 1024), "triangular", 1, True), ((2048, 2048), "triangular", 0, False),
    ((64, 64), "triangular12", 0, False), ((64, 60), "triangular", 0, False), ((64, 750), "square", 1, False),
    ((64, 8), "square", 0, False), ((64, 16), "square", 0, True)], ids=str)
def test_passes_follow_the_object(shape, lattice, dtype, fused):
    kvec = pfc_inputs.lattice_vectors(lattice)

    class Obj:
        x_fused = _x_fused(shape, kvec, dtype)

    assert Obj.x_fused is fused
    assert bench.amplitude_x_passes(Obj(), 4) == (2.5 if fused else 6.0)
