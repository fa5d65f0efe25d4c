"""Slot columns of long documents: worked out in pieces of 8192 rows, the table's state taken from the selection's
checkpoints where these hold every resident (windows up to 4096 keys)."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2508_02124_amd import workloads as wlmod
from paper_2508_02124_amd.device_case import DeviceCase
from test_gpu_parity import check_mask
from test_gpu_slots import scores

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pattern", ["rising", "waves", "random"])
@pytest.mark.parametrize("k,seqlens", [(1, (16385,)), (333, (300, 16385, 0, 24577)), (4096, (20481, 5000)), (4097, (17000,)),
                                       (9000, (33000,)), (18000, (17000, 18001))])
def test_long_documents(gpu, pattern, k, seqlens):
    wl = wlmod.small_workload(f"long_slots_{pattern}_{k}", 37, 2, 1, 64, k, seqlens)
    inp = wlmod.make_inputs(wl)
    print(f"[case] {wl.name} {seqlens}", flush=True)
    case = DeviceCase(inp, gpu, z_override=scores(pattern, wl.H_q, inp.T, k))
    case.mask_gen()
    check_mask(case, wl.name)
    pv = case.plan_views()
    for h in range(wl.H_q):  # a key keeps its column from block to block
        col = np.full(inp.T, -1)
        for bi in range(pv["nblk"]):
            row = pv["slot"][h, bi]
            for keys, at in ((row[row >= 0], np.flatnonzero(row >= 0)), (-2 - row[row < -1], np.flatnonzero(row < -1))):
                seen = col[keys] >= 0
                assert (col[keys][seen] == at[seen]).all(), (h, bi)
                col[keys] = at
