"""Slot columns at their edges: keys that enter a column inside a block of query rows, columns that are
new in the block, keys that enter and expire inside one block, windows wider than the row-wise table."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2508_02124_amd import workloads as wlmod
from paper_2508_02124_amd.device_case import DeviceCase
from test_gpu_parity import check_gradients, check_mask

pytestmark = pytest.mark.gpu


def scores(pattern, H, T, seed):
    rng = np.random.default_rng(seed)
    if pattern == "rising":        # every row admits its key and evicts the oldest: a local band
        z = np.tile(np.linspace(0.1, 1.5, T), (H, 1))
    elif pattern == "falling":     # the first k keys stay for good
        z = np.tile(np.linspace(1.5, 0.1, T), (H, 1))
    elif pattern == "waves":       # bursts of rising scores: keys enter and expire inside one block
        z = 0.5 + 0.4 * np.sin(np.arange(T)[None, :] / (7.0 + 5.0 * np.arange(H)[:, None])) + 1e-3 * rng.random((H, T))
    else:
        z = np.exp(-np.log1p(np.exp(rng.standard_normal((H, T)))))
    return z.astype(np.float32)


@pytest.mark.parametrize("pattern", ["rising", "falling", "waves", "random"])
@pytest.mark.parametrize("d,k,seqlens", [(64, 40, (700, 3)), (128, 255, (257, 900)), (128, 256, (1025,)),
                                         (64, 257, (512, 256, 1)), (128, 300, (299, 301, 640)), (256, 130, (515,))])
def test_slot_sweep_edges(gpu, pattern, d, k, seqlens):
    wl = wlmod.small_workload(f"slots_{pattern}_{d}_{k}", 31, 4, 2, d, k, seqlens)
    inp = wlmod.make_inputs(wl)
    z = scores(pattern, wl.H_q, inp.T, k)
    print(f"[case] {wl.name} {seqlens}", flush=True)
    case = DeviceCase(inp, gpu, z_override=z)
    case.mask_gen()
    check_mask(case, wl.name)
    case.fwd()
    case.bwd()
    check_gradients(case, z.astype(np.float64), "bf16")


@pytest.mark.parametrize("k,n", [(300, 1100), (16400, 17000)])  # the row-wise table, and the wide one
def test_slot_table_names_entering_keys(gpu, k, n):
    """-2 - key: the key enters inside the block, in a column older than the block, and stays to its end."""
    wl = wlmod.small_workload(f"entering_{k}", 33, 2, 1, 64, k, (n,))
    inp = wlmod.make_inputs(wl)
    case = DeviceCase(inp, gpu)
    case.mask_gen()
    check_mask(case, wl.name)
    eg, pv = case.host("expiry"), case.plan_views()
    for h in range(wl.H_q):
        for bi in range(pv["nblk"]):
            r0, r1 = pv["blk"][bi][1:3]
            row = pv["slot"][h, bi]
            named = set((-2 - row[row < -1]).tolist())
            j = np.arange(max(r0, k), max(r1, k))
            j = j[(j < r1) & (eg[h, r0:r1][j - r0] >= r1)] if r1 > k else j[:0]
            stays = set(j.tolist())
            assert named <= stays
            if r0 >= k:            # every column is older than the block
                assert named == stays, (h, bi)
