"""The reference maximum of the forward's online softmax, over score values that random inputs do not have.  The header
is built for the CPU and driven from here."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2508_02124_amd", "csrc")
DRIVER = """
#include "softmax_ref.h"
extern "C" float ref_of(float top, float c2) { return dma::reference_of(top, c2); }
extern "C" float exponent(float s, float c2, float ref) { return dma::weight_exponent(s, c2, ref); }
"""


@pytest.fixture(scope="module")
def ref(tmp_path_factory):
    d = tmp_path_factory.mktemp("softmax_ref")
    (d / "driver.cpp").write_text(DRIVER)
    lib = str(d / "driver.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wno-unused-function", f"-I{CSRC}",
                    str(d / "driver.cpp"), "-o", lib], check=True)
    L = ctypes.CDLL(lib)
    for f, n in ((L.ref_of, 2), (L.exponent, 3)):
        f.argtypes, f.restype = [ctypes.c_float] * n, ctypes.c_float
    return L


SCALES = [float(np.float32(x)) for x in (1.4426950408889634 / np.sqrt(d) for d in (1, 64, 128, 256))]


def test_no_weight_exceeds_one_by_much(ref):
    """For every magnitude of the largest score; and the reference is the rounded product where that is exact enough."""
    r = np.random.default_rng(0)
    tops = [0.0, -0.0] + [float(np.float32(s * m * 2.0 ** e)) for e in range(-20, 127) for m in r.uniform(1, 2, 6)
                          for s in (-1, 1)]
    for c2 in SCALES:
        for top in tops:
            product = np.float32(top) * np.float32(c2)
            got = ref.ref_of(top, c2)
            assert ref.exponent(top, c2, got) <= 1, (top, c2)
            if abs(product) < 2.0 ** 24:
                assert got == product
            elif np.isfinite(product) and abs(product) < 1e38:
                assert abs(got - product) <= abs(float(np.spacing(product)))


def test_reference_of_nothing_is_a_number(ref):
    for c2 in SCALES:
        assert ref.ref_of(float("-inf"), c2) == -np.finfo(np.float32).max
