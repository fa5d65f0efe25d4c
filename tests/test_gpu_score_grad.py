"""Gradient of the content scores at the edges of its row tiles and for every way a group of q-heads is handled."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as orc
from gpu_harness import check_close, tol
from paper_2508_02124_amd import binding as B
from paper_2508_02124_amd import workloads as wlmod

pytestmark = pytest.mark.gpu


EDGES = [(T, *heads) for T in (1, 15, 64, 65, 4099)
         for heads in ((2, 2, 64), (8, 1, 64), (4, 2, 128), (3, 1, 128), (8, 2, 128), (8, 1, 256), (2, 1, 256))]
# 64 channels and a group: on both sides of the row count from which the rows kernel is taken
EDGES += [(T, *heads) for T in (16384, 16385) for heads in ((4, 2, 64), (8, 2, 64), (16, 2, 64))]


@pytest.mark.parametrize("T,H_q,H_kv,d", EDGES)
def test_score_gradient_edges(gpu, T, H_q, H_kv, d):
    print(f"[case] score gradient T={T} {H_q}/{H_kv} d={d}", flush=True)
    r = np.random.default_rng(T + 10 * H_q + d)
    bf = lambda *s: wlmod.bf16_bits_to_f32(wlmod.f32_to_bf16_bits(r.standard_normal(s).astype(np.float32)))
    V, dV0 = bf(T, H_kv, d), bf(T, H_kv, d)
    W = (r.standard_normal((H_q, d)) / np.sqrt(d)).astype(np.float32)
    A = -r.uniform(0.5, 2.0, H_q).astype(np.float32)
    dz = r.standard_normal((H_q, T)).astype(np.float32)
    dev = lambda x, dt=torch.float32: torch.from_numpy(np.ascontiguousarray(x)).to(gpu).to(dt)
    shape = B.make_shape(T=T, n_docs=1, H_q=H_q, H_kv=H_kv, d=d, k=1)
    rW, rA, rV = orc.mask_backward(V, W, A, dz, H_q)
    for accumulate in (False, True):
        dW, dA, dV = torch.full((H_q, d), 7.0, device=gpu), torch.full((H_q,), 7.0, device=gpu), dev(dV0, torch.bfloat16)
        B.dma_mask_bwd(shape, dev(V, torch.bfloat16), dev(W), dev(A), dev(dz), dW, dA, dV, accumulate)
        # fp32 sums of up to T terms of size one: rounding of about sqrt(T) 2^-24 per sum, far below 1e-4 of it
        check_close("dW", dW.cpu().numpy(), rW, atol=1e-4 * np.sqrt(T), rtol=1e-4, frob=1e-5)
        check_close("dA", dA.cpu().numpy(), rA, atol=1e-4 * np.sqrt(T), rtol=1e-4, frob=1e-5)
        check_close("dVz", dV.float().cpu().numpy(), rV + (dV0 if accumulate else 0), **tol(True))
