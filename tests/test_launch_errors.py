"""A launch that fails is reported, whichever launch of a call it is.  The library is loaded over a stand-in for the runtime's
launch functions, which runs nothing and lets the n-th launch fail (no GPU needed); in a process of its own, so that no
other test meets the stand-in."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2508_02124_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <cstddef>
struct dim3 { unsigned x, y, z; };
static int launches, failing, last;
extern "C" {
void start(int n) { launches = last = 0; failing = n; }
int launched() { return launches; }
int __hipPushCallConfiguration(dim3, dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
  *grid = *block = {1, 1, 1};
  *lds = 0;
  *stream = nullptr;
  return 0;
}
int hipLaunchKernel(const void*, dim3, dim3, void**, size_t, void*) { return ++launches == failing ? last = 719 : 0; }
int hipGetLastError() { const int e = last; last = 0; return e; }
}
"""

# The calls of a step, at shapes that take each of the selection's routes: by blocks, with checkpoints and slot pieces, sorted
# (short and long segments), not causal, every key kept.
CALLS = r"""
import ctypes, sys
runtime = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2508_02124_amd import binding as B
P = 0x1000  # (never dereferenced: nothing runs)
seen = set()
for T, k, causal, H_q in ((8192, 64, True, 2), (65536, 64, True, 4), (65536, 20000, True, 2), (200000, 64, True, 3), (4096, 64, False, 2),
                          (1000, 2000, True, 2)):
    shape = B.make_shape(T=T, n_docs=1, H_q=H_q, H_kv=1, d=64, k=k, causal=causal)
    calls = {
        "mask_gen": lambda: B.dma_mask_gen(shape, P, P, P, P, P, P, P, P, stream=0),
        "mask_gen, scores given": lambda: B.dma_mask_gen(shape, P, None, None, P, P, P, None, P, stream=0),
        "fwd": lambda: B.dma_fwd(shape, *[P] * 9, None, 0, stream=0),
        "bwd_scores": lambda: B.dma_bwd_scores(shape, *[P] * 19, 1 << 40, stream=0),
    }
    for name, call in calls.items():
        runtime.start(0)
        call()
        n = runtime.launched()
        assert n > 0
        seen.add((name, n))
        for i in range(1, n + 1):
            runtime.start(i)
            try:
                call()
                print(f"LOST: {name} T={T} k={k} causal={causal}, launch {i} of {n}")
            except B.DmaError as e:
                assert e.status == B.DMA_EHIP, (name, i, e)
print("calls", len(seen))
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_failed_launch_is_reported(tmp_path):
    if not os.path.exists(B.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    source, stand_in, calls = tmp_path / "stand_in.cpp", tmp_path / "stand_in.so", tmp_path / "calls.py"
    source.write_text(STAND_IN)
    calls.write_text(CALLS)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", str(source), "-o", str(stand_in)], check=True)
    r = subprocess.run([sys.executable, str(calls), str(stand_in), ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "LOST" not in r.stdout and "calls" in r.stdout, r.stdout
