"""Host rules of spatially sorted frames, compiled for the CPU from the
library's own header: where a point lies (the cell and the place in it name one
image, also for points on a cell face)."""
import ctypes
import math
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

from paper_1808_01478_amd import build

SOURCE = """
#include "dh_internal.h"
extern "C" double wrap_cell(double f, unsigned int *place) { return dh::wrap_cell(f, *place); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    (d / "rules.cpp").write_text(SOURCE)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc())))
    subprocess.run([build.hipcc(), *build.CPU_FLAGS, "-shared", "-D__HIP_PLATFORM_AMD__",
                    f"-I{rocm}/include", f"-I{build.INCLUDE}", f"-I{build.CSRC}",
                    str(d / "rules.cpp"), "-o", str(d / "rules.so")], check=True)
    so = ctypes.CDLL(str(d / "rules.so"))
    so.wrap_cell.argtypes = [ctypes.c_double, ctypes.POINTER(ctypes.c_uint)]
    so.wrap_cell.restype = ctypes.c_double
    return so


def near_faces():
    """Fractional coordinates on and next to integers, from both sides."""
    out = [0.0, -0.0, 5e-324, -5e-324, -1e-300]
    for k in range(30, 60):
        out += [math.ldexp(1.0, -k), -math.ldexp(1.0, -k)]
    for n in (-1000, -3, -2, -1, 0, 1, 2, 7, 1000):
        f = float(n)
        for _ in range(3):
            out += [f]
            f = math.nextafter(f, math.inf)
        f = float(n)
        for _ in range(3):
            f = math.nextafter(f, -math.inf)
            out += [f]
    rng = np.random.Generator(np.random.PCG64(3))
    return out + list(rng.uniform(-3.0, 4.0, 500))


def test_cell_and_place_name_one_image(lib):
    for f in near_faces():
        place = ctypes.c_uint()
        n = lib.wrap_cell(f, ctypes.byref(place))
        assert n == math.floor(n)
        # the place read back is below the exact f - n by less than its unit
        # (2^-32) and the rounding of the difference (2^-53)
        gap = Fraction(f) - Fraction(n) - Fraction(place.value, 1 << 32)
        assert -Fraction(1, 1 << 53) <= gap < Fraction(1, 1 << 32), (f, n, place.value)
