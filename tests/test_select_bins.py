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
extern "C" int bins_of(float top, float low, const float* z, int n, uint32_t* out) {
  const B b = made(top, low);
  if (b.ok) for (int i = 0; i < n; i++) out[i] = b.of(z[i]);
  return b.ok;
}
extern "C" uint32_t bound(float top, float low, int bin, int cut) { return made(top, low).bound(bin, cut); }
extern "C" int behind(float top, float low, float z) { return made(top, low).behind(z); }
extern "C" int between(float top, float low, int b0, int b1, float z) {
  const B b = made(top, low);
  return z + b.add <= b.most(b0) && z + b.add >= b.least(b1);
}
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
    L.bins_of.argtypes = [f, f, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    L.bound.argtypes, L.bound.restype = [f, f, ctypes.c_int, ctypes.c_int], ctypes.c_uint32
    L.behind.argtypes, L.between.argtypes = [f, f, f], [f, f, ctypes.c_int, ctypes.c_int, f]
    L.key.argtypes, L.key.restype = [f], ctypes.c_uint32
    L.value.argtypes, L.value.restype = [ctypes.c_uint32], f
    return L


def bins_of(lib, top, low, z):
    z, out = np.ascontiguousarray(z, dtype=np.float32), np.empty(len(z), dtype=np.uint32)
    return out.astype(np.int64) if lib.bins_of(top, low, z.ctypes.data, len(z), out.ctypes.data) else None


def ranges(rng):
    """(top, low, scores in descending order): of every size and sign, bins over all of the scores or over a part of them."""
    special = np.array([0.0, -0.0, 1e-45, -1e-45, 1e-38, -1e-38, 1, -1, 1 + 2.0 ** -23, 3e38, -3e38, 1e30, -1e30], dtype=np.float32)
    beyond = np.array([np.inf, -np.inf, 3.4e38, -3.4e38, 0.0, -1e-44], dtype=np.float32)
    for trial in range(400):
        spread = np.float32(10.0 ** rng.uniform(-44, 38))
        z = rng.standard_normal(200).astype(np.float32) * spread + np.float32(rng.choice([0, 0, 1, -1, 1000, -1e6]))
        z = np.concatenate([z if trial % 3 else np.abs(z), special[rng.integers(0, len(special), trial % 4)]]).astype(np.float32)
        z = -np.sort(-z[np.isfinite(z)])
        cut = trial % 5 * len(z) // 10
        yield float(z[cut // 4]), float(z[len(z) - 1 - cut]), -np.sort(-np.concatenate([z, beyond]))
    for top, low in ((1.0, 0.5), (1e-38, 1e-42), (1e-42, 1e-44), (3e-34, 0.0), (1e-38, -1e-44), (1e-40, -1e-40), (3e38, 1e38)):
        yield top, low, -np.sort(-np.concatenate([beyond, -beyond[2:], np.array([top, low], dtype=np.float32)]))


def test_bins_never_fall_and_bounds_are_theirs(lib):
    binned = 0
    for top, low, z in ranges(np.random.default_rng(0)):
        b = bins_of(lib, top, low, z)
        if b is None:
            continue
        binned += 1
        assert (np.diff(b) >= 0).all() and b[0] == 0 and b[-1] < lib.bins(), (top, low)
        assert bins_of(lib, top, low, [top])[0] == 0 and bins_of(lib, top, low, [low])[0] == b[-1]
        behind = np.array([lib.behind(top, low, x) for x in z])
        assert not behind[z >= low].any() and (np.diff(behind) >= 0).all() and (b[behind == 1] == b[-1]).all()
        some = sorted({0, 1, int(b[50 % len(b)]), int(b[-1])})
        for bin in some + [int(b[-1]) + 1]:
            for cut in (0, 1):
                k = lib.bound(top, low, bin, cut)
                for key, before in ((k, False), (k - 1, True)):
                    if lib.key(np.inf) <= key <= lib.key(-np.inf):
                        x = lib.value(key)
                        assert (bins_of(lib, top, low, [x])[0] < bin and not (cut and lib.behind(top, low, x))) == before
        for b0 in some:
            for b1 in some:
                assert [bool(lib.between(top, low, b0, b1, x)) for x in z] == list((b >= b0) & (b <= b1)), (top, low, b0, b1)
    assert binned > 250


def test_what_is_not_a_number_has_a_bin(lib):
    quiet = np.array([0x7FC00000, 0xFFC00000, 0x7F800001, 0xFF800001], dtype=np.uint32).view(np.float32)
    b = bins_of(lib, 1.0, 0.25, quiet)
    assert (b >= 0).all() and (b < lib.bins()).all()


@pytest.mark.parametrize("top,low", [(1.0, 1.0), (0.5, 1.0), (np.inf, 0.0), (1.0, -np.inf), (3e38, -3e38),
                                     (0.0, -0.0), (np.nan, np.nan)])
def test_scores_without_bins(lib, top, low):
    assert bins_of(lib, top, low, [0.0]) is None


def scores(gate, spread, n, rng):
    return np.exp(gate * np.logaddexp(0, spread * rng.standard_normal(n))).astype(np.float32)


@pytest.mark.parametrize("n,k", [(16384, 2048), (4369, 512)])
@pytest.mark.parametrize("gate,spread,odd", [(-8, 1, None), (-2, 1, None), (-0.5, 1, None), (0.5, 1, None), (2, 1, None), (4, 1, None),
                                             (-2, 3, None), (1, 3, None), (6, 3, None), (-1, 1, 1e30), (-1, 1, 0.0), (-1, 1, -np.inf)])
def test_blocks_of_gated_scores_are_ranked_by_bins(lib, gate, spread, odd, n, k):
    """The keys in the bins of ranks k - e to k are not many more than a block of 256 rows has to rank, but for a few blocks."""
    rng = np.random.default_rng(1)
    z = scores(gate, spread, n, rng)
    if odd is not None:  # outliers, zeros, masked keys
        z[rng.random(n) < (0.1 if odd == -np.inf else 2e-4)] = odd
    blocks = beyond = 0
    for lo in range((k + 255) // 256 * 256, n - 256, 256):
        old, kept = z[:lo], min(k, lo)
        sample = old[np.arange(256) * lo // 256]
        sample = sample[np.isfinite(sample) & (sample != 0)]
        top, low = float(sample.max()), float(sample.min())
        counts = np.bincount(bins_of(lib, top, low, old), minlength=lib.bins())
        ends = np.cumsum(counts)
        last = np.searchsorted(ends, kept - 1, "right") if kept < lo else lib.bins() - 1
        e = int((bins_of(lib, top, low, z[lo:lo + 256]) <= last).sum())
        rank = max(0, kept - min(e, lo + 256 - k))
        first = np.searchsorted(ends, rank, "right")
        blocks += 1
        beyond += ends[last] - ends[first] + counts[first] - (kept - rank) > lib.near()
    assert beyond <= blocks // 8, (beyond, blocks)
