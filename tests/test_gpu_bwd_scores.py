"""dma_bwd_scores (the backward of a whole step) against the oracle, and against dma_bwd followed by dma_mask_bwd."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2508_02124_amd import binding as B
from paper_2508_02124_amd import workloads as wlmod
from gpu_harness import DeviceCase, check_close, tol

pytestmark = pytest.mark.gpu


def forward(gpu, H_q, H_kv, d, lens, k, dtype="bf16", z=None):
    wl = wlmod.small_workload(f"bwd_scores_{d}", 300 + k, H_q, H_kv, d, k, lens)
    case = DeviceCase(wlmod.make_inputs(wl, dtype=dtype), gpu, z_override=z)
    case.mask_gen()
    case.fwd()
    return case


def scores_bwd(c):
    dW, dA = (torch.full_like(x, float("nan")) for x in (c.W, c.A))
    B.dma_bwd_scores(c.shape, c.Q, c.K, c.V, c.O, c.dO, c.LSE, c.z, c.expiry, c.mask, c.cu, c.W, c.A, c.dQ, c.dK, c.dV,
                     c.dz, dW, dA, c.ws, c.ws_bytes)
    return dW, dA


# (3 and 5 q-heads per kv-head, and fp32: the two calls' kernels)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H_q,H_kv,d", [(2, 2, 64), (4, 2, 64), (4, 1, 64), (8, 1, 64), (3, 1, 64), (3, 3, 128), (4, 2, 128),
                                        (4, 1, 128), (8, 1, 128), (5, 1, 128), (2, 2, 256), (4, 1, 256)])
def test_against_the_oracle(gpu, H_q, H_kv, d, dtype):
    for lens, k in (((1, 33, 64), 10), ((300, 17), 65)):
        print(f"[case] bwd_scores {H_q}/{H_kv} d={d} {dtype} {lens} k={k}", flush=True)
        c = forward(gpu, H_q, H_kv, d, lens, k, dtype)
        dW, dA = scores_bwd(c)
        inp = c.inp
        dQ, dK, dV, dz = orc.dma_backward(inp.Q, inp.K, inp.V, c.host("z").astype(np.float64), inp.dO, inp.cu_seqlens, k,
                                          O_stored=c.host("O"), LSE_stored=c.host("LSE"))
        # the chain rule's own rounding: from the dz that the call returned
        rW, rA, rVz = orc.mask_backward(inp.V, inp.W, inp.A, c.host("dz"), H_q)
        t = tol(dtype == "bf16")
        for name, ref in (("dQ", dQ), ("dK", dK), ("dV", np.asarray(dV) + np.asarray(rVz)), ("dz", dz)):
            check_close(name, c.host(name), ref, **t)
        t32 = dict(atol=1e-4, rtol=1e-4, frob=1e-5)  # fp32 sums of about 300 terms
        check_close("dW", dW.cpu().numpy(), rW, **t32)
        check_close("dA", dA.cpu().numpy(), rA, **t32)


# Enough rows for the form that does not read rows that no head keeps (at random scores), with odd ends.
@pytest.mark.parametrize("kind", ["random", "rising"])
@pytest.mark.parametrize("H_q,H_kv,d,lens,k", [(4, 4, 64, (5000, 6001, 5555), 200), (4, 2, 128, (9001, 7777), 150),
                                               (4, 1, 256, (10007, 6500), 100)])
def test_against_the_two_calls(gpu, H_q, H_kv, d, lens, k, kind):
    print(f"[case] bwd_scores {H_q}/{H_kv} d={d} {kind} {lens}", flush=True)
    T = sum(lens)
    rng = np.random.default_rng(5)
    z = np.tile(np.linspace(0.1, 1, T), (H_q, 1)) if kind == "rising" else rng.uniform(0.1, 1, (H_q, T))
    c = forward(gpu, H_q, H_kv, d, lens, k, z=z)
    c.bwd()
    part = c.dV.float().clone()
    dW2, dA2 = torch.empty_like(c.W), torch.empty_like(c.A)
    B.dma_mask_bwd(c.shape, c.V, c.W, c.A, c.dz, dW2, dA2, c.dV, True)
    two = {name: getattr(c, name).float().clone() for name in ("dQ", "dK", "dV", "dz")}
    for name in ("dQ", "dK", "dV", "dz"):
        getattr(c, name).fill_(float("nan"))
    dW, dA = scores_bwd(c)
    # fp32 sums in another order: 2e-5 of the largest value.  bf16 has 8 significant bits: two sums that close may round to
    # neighbouring values, up to 2^-7 of the value apart; the attention's part of dV is rounded once more by the two calls,
    # by up to 2^-8 of it.
    for name, ref in two.items():
        got = getattr(c, name).float()
        place = 2.0 ** -7 if name != "dz" else 0.0
        bound = place * ref.abs() + (2.0 ** -8 * part.abs() if name == "dV" else 0.0) + 2e-5 * ref.abs().max()
        beyond = int(((got - ref).abs() > bound).sum()) + int(torch.isnan(got).sum())
        assert beyond == 0, (name, beyond)
    for got, ref in ((dW, dW2), (dA, dA2)):
        assert float((got - ref).abs().max()) <= 2e-5 * float(ref.abs().max())


# Gates above 128, for which the score of a value of zeros is beyond fp32, with values whose scores are not: rows that no head
# keeps are not read and take no part.
@pytest.mark.parametrize("H_q,H_kv,d,lens,k", [(4, 4, 64, (16500,), 200), (4, 2, 128, (9001, 7777), 150),
                                               (4, 1, 256, (10007, 6500), 100)])
def test_gates_beyond_the_range(gpu, H_q, H_kv, d, lens, k):
    print(f"[case] bwd_scores {H_q}/{H_kv} d={d} gates of 129 to 200 {lens}", flush=True)
    inp = wlmod.make_inputs(wlmod.small_workload(f"gates_{d}", 400 + k, H_q, H_kv, d, k, lens))
    inp.A[:] = np.linspace(129, 200, H_q)
    inp.W *= 0.5
    inp.W[:, 0] = -6
    inp.V[:, :, 0] = 1  # x about -6 +- 0.5: scores of 1.04 to 280
    inp.bits["V"] = wlmod.f32_to_bf16_bits(inp.V)
    c = DeviceCase(inp, gpu)
    c.mask_gen()
    c.fwd()
    c.bwd()
    part = c.host("dV")
    dW, dA = scores_bwd(c)
    dz = c.host("dz")
    assert (dz == 0).mean() > 0.3  # (there are rows that no head keeps)
    rW, rA, rVz = orc.mask_backward(inp.V, inp.W, inp.A, dz, H_q)
    # x: an fp32 sum of products whose sizes add up to about 16, in 13 roundings: error up to 16 * 13 * 2^-24 = 1.3e-5; a score's
    # relative error is up to 200 * sigmoid(-3.6) = 5.5 times that, 7e-5, and the sums' own 1e-5: 1e-4 of the terms' sizes
    sizes = np.zeros(rVz.shape)
    for h in range(H_q):
        v = inp.V[:, h // (H_q // H_kv)].astype(np.float64)
        x = v @ inp.W[h].astype(np.float64)
        sp = np.log1p(np.exp(x))
        weight = np.abs(dz[h]) * np.exp(inp.A[h] * sp)
        assert abs(dA[h].item() - rA[h]) <= 1e-4 * (weight * sp).sum()
        mass = (weight * inp.A[h] / (1 + np.exp(-x))) @ np.abs(v)
        assert (np.abs(dW[h].cpu().numpy() - rW[h]) <= 1e-4 * mass).all()
        sizes[:, h // (H_q // H_kv)] += np.outer(weight * inp.A[h] / (1 + np.exp(-x)), np.abs(inp.W[h]))
    # the attention's part comes from dma_bwd, which rounds it to bf16 (2^-9 of it), and the sum, which may cancel, is rounded too
    ref, got = part + rVz, c.host("dV")
    assert (np.abs(got - ref) <= 2.0 ** -8 * (np.abs(ref) + np.abs(part)) + 1e-4 * sizes + 1e-4).all()
