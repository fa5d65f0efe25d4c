"""Calls of few blocks, whose half blocks are worked out by two waves for every 32 rows (each with its own units of the
tiles), at the edges of tiles, units and blocks and on both sides of the rule that chooses this form (all half blocks fit
the 256 compute units); documents of which one wave of a pair keeps nothing, and scores that climb, so that the two
waves' statistics differ widely."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as orc
from paper_2508_02124_amd import workloads as wlmod
from gpu_harness import DeviceCase, check_close, tol
from test_gpu_parity import check_gradients

pytestmark = pytest.mark.gpu


def run(gpu, H_q, H_kv, d, lens, k, climb=0.0):
    inp = wlmod.make_inputs(wlmod.small_workload(f"parts_{d}_{k}", 700 + k, H_q, H_kv, d, k, lens))
    if climb:  # a factor of exp(climb) from one unit of 32 keys to the next, up and down
        j = np.arange(inp.T)
        inp.Q[:] = wlmod.bf16_bits_to_f32(wlmod.f32_to_bf16_bits(0.25 * inp.Q + 1))
        step = climb * (j // 32 % 3) / np.sqrt(d)
        inp.K[:] = wlmod.bf16_bits_to_f32(wlmod.f32_to_bf16_bits(0.25 * inp.K + step[:, None, None].astype(np.float32)))
        for x in ("Q", "K"):
            inp.bits[x] = wlmod.f32_to_bf16_bits(getattr(inp, x))
    case = DeviceCase(inp, gpu)
    case.mask_gen()
    case.fwd()
    heads = sorted({0, H_q - 1})
    O, LSE = orc.dma_forward(inp.Q, inp.K, inp.V, case.host("z"), inp.cu_seqlens, k, heads=heads)[:2]
    check_close(f"O d={d} k={k}", case.host("O")[:, heads], np.asarray(O)[:, heads], **tol(True))
    check_close(f"LSE d={d} k={k}", case.host("LSE")[heads], np.asarray(LSE)[heads], **tol(True))
    return case, inp


@pytest.mark.parametrize("climb", [0.0, 6.0], ids=["plain", "climbing"])
@pytest.mark.parametrize("lens", [(1, 31, 32, 33, 63, 64, 65), (127, 129, 257), (600,)], ids=str)
@pytest.mark.parametrize("d", [64, 128])
def test_forward(gpu, d, lens, climb):
    for k in (1, 31, 32, 33, 64, 65, 200, 1024):
        print(f"[case] forward d={d} documents {lens} k={k}", flush=True)
        run(gpu, 2, 1, d, lens, k, climb)


# 16 heads x 8 blocks: all half blocks find a compute unit; 16 x 9: they do not
@pytest.mark.parametrize("T", [2048, 2049])
@pytest.mark.parametrize("d", [64, 128])
def test_both_sides_of_the_rule(gpu, d, T):
    print(f"[case] forward d={d} T={T}", flush=True)
    run(gpu, 16, 4, d, (T,), 300)


@pytest.mark.parametrize("lens", [(33, 65, 129, 257), (600,)], ids=str)
def test_gradients(gpu, lens):
    for k in (31, 64, 65, 200, 1024):
        print(f"[case] gradients documents {lens} k={k}", flush=True)
        case, inp = run(gpu, 2, 1, 128, lens, k)
        case.bwd()
        check_gradients(case, case.host("z").astype(np.float64), "bf16", label=f"k={k} ")
