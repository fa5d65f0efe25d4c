"""The bins of the selection by blocks, over scores that random inputs do not have and over scores of gates of either sign.
The header is built for the CPU and driven from here."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2508_02124_amd", "csrc")
DRIVER = """
#include "select_bins.h"
using namespace dma;
using B = Bins<BIN_BITS>;
static B made(float top, float low) { B b; b.init(desc_key(top), desc_key(low)); return b; }
extern "C" int bins_of(float top, float low, const float* z, int n, int any, uint32_t* out) {
  const B b = made(top, low);
  if (b.ok) for (int i = 0; i < n; i++) out[i] = any ? b.of_any(z[i]) : b.of_behind(z[i]);
  return b.ok;
}
extern "C" uint32_t bound(float top, float low, int bin) { return made(top, low).bound(bin); }
extern "C" uint32_t key(float z) { return desc_key(z); }
extern "C" float value(uint32_t k) { return key_value(k); }
extern "C" int bins() { return 1 << BIN_BITS; }
extern "C" int near() { return NEAR; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("select_bins")
    (d / "driver.cpp").write_text(DRIVER)
    path = str(d / "driver.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(d / "driver.cpp"), "-o", path], check=True)
    L, f = ctypes.CDLL(path), ctypes.c_float
    L.bins_of.argtypes = [f, f, ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    L.bound.argtypes, L.bound.restype = [f, f, ctypes.c_int], ctypes.c_uint32
    L.key.argtypes, L.key.restype = [f], ctypes.c_uint32
    L.value.argtypes, L.value.restype = [ctypes.c_uint32], f
    return L


def bins_of(lib, top, low, z, any=True):
    z, out = np.ascontiguousarray(z, dtype=np.float32), np.empty(len(z), dtype=np.uint32)
    return out.astype(np.int64) if lib.bins_of(top, low, z.ctypes.data, len(z), any, out.ctypes.data) else None


def test_bins_never_fall_and_bounds_are_theirs(lib):
    rng = np.random.default_rng(0)
    special = np.array([0.0, -0.0, 1e-45, -1e-45, 1e-38, -1e-38, 1, -1, 1 + 2.0 ** -23, 3e38, -3e38, 1e30, -1e30], dtype=np.float32)
    binned = 0
    for trial in range(400):
        spread = np.float32(10.0 ** rng.uniform(-44, 38))
        z = rng.standard_normal(200).astype(np.float32) * spread + np.float32(rng.choice([0, 0, 1, -1, 1000, -1e6]))
        z = np.concatenate([z if trial % 3 else np.abs(z), special[rng.integers(0, len(special), trial % 4)]]).astype(np.float32)
        z = z[np.isfinite(z)]
        top, low = float(z.max()), float(z.min())
        beyond = np.array([np.inf, -np.inf, 3.4e38, -3.4e38], dtype=np.float32)  # (clamped: new scores may lie outside)
        z = -np.sort(-np.concatenate([z, beyond]))
        b = bins_of(lib, top, low, z)
        if b is None:
            continue
        binned += 1
        assert (np.diff(b) >= 0).all() and b[0] == 0 and b[-1] < lib.bins(), (top, low)
        # a range that leaves the worst out: these come behind its last bin, or share it
        middle = float(z[len(z) // 2])
        if (part := bins_of(lib, top, middle, z[2:-2], any=False)) is not None:
            inside = z[2:-2] >= middle
            assert (part[inside] < lib.bins()).all() and (part[~inside] >= part[inside].max()).all(), (top, middle)
        for bin in {0, 1, int(b[50]), int(b[-1]), int(b[-1]) + 1}:
            k = lib.bound(top, low, bin)
            assert k >= lib.key(top) and (k <= lib.key(low) or bin > b[-1])
            if bin <= b[-1]:
                assert bins_of(lib, top, low, [lib.value(k)])[0] >= bin
            else:
                assert k == lib.key(low) + 1
            if k > lib.key(top):
                assert bins_of(lib, top, low, [lib.value(k - 1)])[0] < bin
    assert binned > 300


def test_scores_far_behind_the_range(lib):
    far = np.array([-1e-44, -1e-38, -1.0, -1e30, -3.4e38], dtype=np.float32)
    for top, low in ((1.0, 0.5), (1e-38, 1e-42), (1e-42, 1e-44), (3e-34, 0.0), (1e-38, -1e-44), (1e-40, -1e-40), (2.0, -1e-3), (3e38, 1e38)):
        last, behind = bins_of(lib, top, low, [low])[0], far[far < low]
        b = bins_of(lib, top, low, behind, any=False)
        assert (b >= last).all() and (np.diff(b) >= 0).all(), (top, low, b, last)


@pytest.mark.parametrize("top,low", [(1.0, 1.0), (np.inf, 0.0), (1.0, -np.inf), (3e38, -3e38), (0.0, -0.0), (np.nan, np.nan)])
def test_scores_without_bins(lib, top, low):
    assert bins_of(lib, top, low, [0.0]) is None


def scores(gate, spread, n, rng):
    return np.exp(gate * np.logaddexp(0, spread * rng.standard_normal(n))).astype(np.float32)


@pytest.mark.parametrize("n,k", [(16384, 2048), (4369, 512)])
@pytest.mark.parametrize("gate,spread", [(-8, 1), (-2, 1), (-0.5, 1), (0.5, 1), (1, 1), (2, 1), (4, 1), (6, 1), (-2, 3), (1, 3)])
def test_blocks_of_gated_scores_are_ranked_by_bins(lib, gate, spread, n, k):
    """The keys in the bins of ranks k - e to k are not many more than a block of 256 rows has to rank, but for a few blocks."""
    z = scores(gate, spread, n, np.random.default_rng(1))
    blocks = beyond = 0
    for lo in range((k + 255) // 256 * 256, n - 256, 256):
        old, kept = z[:lo], min(k, lo)
        top, low = float(old.max()), float(old.min())
        counts = np.bincount(bins_of(lib, top, low, old), minlength=lib.bins())
        ends = np.cumsum(counts)
        last = np.searchsorted(ends, kept - 1, "right") if kept < lo else lib.bins() - 1
        e = int((bins_of(lib, top, low, z[lo:lo + 256]) <= last).sum())
        rank = max(0, kept - min(e, lo + 256 - k))
        first = np.searchsorted(ends, rank, "right")
        blocks += 1
        beyond += ends[last] - ends[first] + counts[first] - (kept - rank) > lib.near()
    assert beyond <= blocks // 8, (beyond, blocks)
