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
extern "C" float none() { return dma::REF_NONE; }
extern "C" float limit() { return __builtin_bit_cast(float, dma::SUM_LIMIT); }
"""


@pytest.fixture(scope="module")
def ref(tmp_path_factory):
    d = tmp_path_factory.mktemp("softmax_ref")
    (d / "driver.cpp").write_text(DRIVER)
    lib = str(d / "driver.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wno-unused-function", f"-I{CSRC}",
                    str(d / "driver.cpp"), "-o", lib], check=True)
    L = ctypes.CDLL(lib)
    for f, n in ((L.ref_of, 2), (L.exponent, 3), (L.none, 0), (L.limit, 0)):
        f.argtypes, f.restype = [ctypes.c_float] * n, ctypes.c_float
    return L


SCALES = [float(np.float32(x)) for x in (1.4426950408889634 / np.sqrt(d) for d in (1, 64, 128, 256))]


def test_no_weight_overflows(ref):
    """For every magnitude of the largest score; and the reference is the rounded product where its weight does not."""
    r = np.random.default_rng(0)
    tops = [0.0, -0.0] + [float(np.float32(s * m * 2.0 ** e)) for e in range(-20, 127) for m in r.uniform(1, 2, 6)
                          for s in (-1, 1)]
    for c2 in SCALES:
        for top in tops:
            product = np.float32(top) * np.float32(c2)
            got = ref.ref_of(top, c2)
            assert ref.exponent(top, c2, got) <= 100, (top, c2)
            if np.isfinite(product) and abs(product) < 1e38:
                assert abs(got - product) <= abs(float(np.spacing(product)))
                if abs(product) < 2.0 ** 31 or ref.exponent(top, c2, product) <= 100:   # (half of a last place: at most 64)
                    assert got == product


def test_reference_of_nothing_is_a_number(ref):
    for c2 in SCALES:
        assert ref.ref_of(float("-inf"), c2) == -np.finfo(np.float32).max


def test_a_row_that_has_kept_nothing_forms_no_nan(ref):
    """Masked scores get no weight, and every other score is either seen as too large or weighted as the maximum."""
    for c2 in SCALES:
        assert ref.exponent(float("-inf"), c2, ref.none()) == float("-inf")
        for score in [s * m * 2.0 ** e for e in range(-60, 127) for m in (1, 1.7) for s in (-1, 1)] + [0.0]:
            x = ref.exponent(score, c2, ref.none())
            assert not np.isnan(x)
            if score * c2 > -np.finfo(np.float32).max:   # (below: beyond the range of the exponents, a mask)
                assert x > np.log2(ref.limit()), (c2, score)


def softmax_row(ref, scores, c2, unit=16):
    """l and the reference after the steps of the forward: `unit` scores at a time, the first 64 always through the
    maximum."""
    f32 = np.float32
    m, l = f32(ref.none()), f32(0)
    for i in range(0, len(scores), unit):
        s = scores[i:i + unit]
        with np.errstate(over="ignore"):
            weights = lambda: np.exp2(np.array([ref.exponent(x, c2, m) for x in s], dtype=np.float32))
            total = weights().sum(dtype=np.float32)
            assert not np.isnan(total)
            if total > (0 if i < 64 else ref.limit()):
                top = f32(ref.ref_of(max(s), c2))
                if top > m:
                    l, m = f32(l * np.exp2(m - top)), top
                total = weights().sum(dtype=np.float32)
        l = f32(l + total)
        assert np.isfinite(l)
    return l, m


@pytest.mark.parametrize("seed", range(8))
def test_rows_of_every_kind_of_score(ref, seed):
    """Rows that begin with masked keys (-inf, or a large finite bias), climb by more than the limit, or hold both: log2 of
    the sum of weights against 64 bits.  Tolerance: the exponents' rounding, c2 |score| 2^-24 each, and l's, 64 * 2^-24."""
    r = np.random.default_rng(seed)
    inf = float("inf")
    for c2 in SCALES:
        for _ in range(60):
            n = int(r.integers(1, 260))
            s = r.standard_normal(n) * r.choice([1, 30, 300])
            s += r.choice([0, 1]) * np.cumsum(r.random(n) * r.choice([1, 20]))
            n_masked = int(r.integers(0, n))
            s[:n_masked] = r.choice([-inf, -1e10, -3e12, -1e30, -3e37, -3.4e38])
            s[n_masked:][r.random(n - n_masked) < 0.2] = r.choice([-inf, -1e30])
            s[int(r.integers(n_masked, n))] = r.standard_normal()
            s = s.astype(np.float32)
            l, m = softmax_row(ref, [float(x) for x in s], c2)
            real = s[s > -1e9].astype(np.float64) * c2
            want = real.max() + np.log2(np.exp2(real - real.max()).sum())
            assert abs(float(m) + np.log2(float(l)) - want) <= 2.0 ** -22 * np.abs(real).max() + 2.0 ** -16
