"""The one-launch selection of a decode and the grouped gather behind it, at the sizes where they change path:
keys per wave (multiples of 1024), the register capacities (16384 and 65536 keys), the candidate limits
(512 ranked, 8192 listed, more = counted from all keys), ties across the threshold, scores of every sign, and
numbers of (sequence, kv-head) pairs that 8 does not divide."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle as orc
from gpu_harness import check_close, tol
from paper_2508_02124_amd import binding as B
from paper_2508_02124_amd import workloads as wlmod

pytestmark = pytest.mark.gpu


def scores(pattern, H, T, rng):
    if pattern == "ordinary":
        return np.exp(-np.log1p(np.exp(rng.standard_normal((H, T))))).astype(np.float32)
    if pattern == "equal":
        return np.full((H, T), 0.5, np.float32)
    if pattern == "levels":                       # heavy ties
        return (np.round(rng.random((H, T)) * 24) / 24).astype(np.float32)
    if pattern == "outlier":                      # one far value: nearly all keys share a few bins
        z = (0.5 + 1e-3 * rng.random((H, T))).astype(np.float32)
        z[:, T // 3] = 1e-30
        return z
    if pattern == "signed":
        z = rng.standard_normal((H, T)).astype(np.float32)
        z[:, ::7] = 0.0
        z[:, 3::7] = -0.0
        return z
    return np.tile(np.linspace(0.1, 0.9, T), (H, 1)).astype(np.float32)  # "rising": the kept keys are one wave's


def decode(gpu, lens, H_q, H_kv, d, k, z, rng, max_seqlen=0):
    T, n_docs = sum(lens), len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rb = lambda *s: wlmod.bf16_bits_to_f32(wlmod.f32_to_bf16_bits(rng.standard_normal(s).astype(np.float32)))
    q, K, V = rb(n_docs, H_q, d), rb(T, H_kv, d), rb(T, H_kv, d)
    dev = lambda x, dt: torch.from_numpy(np.ascontiguousarray(x)).to(gpu).to(dt)
    shape = B.make_shape(T=T, n_docs=n_docs, H_q=H_q, H_kv=H_kv, d=d, k=k, max_seqlen=max_seqlen)
    nb, kcap = B.dma_decode_kept_bytes(shape), min(k, T)
    kept = torch.full((nb // 4,), -7, dtype=torch.int32, device=gpu)
    o = torch.full((n_docs, H_q, d), float("nan"), dtype=torch.bfloat16, device=gpu)
    lse = torch.full((H_q, n_docs), float("nan"), device=gpu)
    B.dma_decode(shape, dev(q, torch.bfloat16), dev(K, torch.bfloat16), dev(V, torch.bfloat16), dev(z, torch.float32),
                 dev(cu, torch.int32), o, lse, kept, nb)
    got = kept.cpu().numpy()[: n_docs * H_q * kcap].reshape(n_docs, H_q, kcap)
    return q, K, V, cu, got, o.float().cpu().numpy(), lse.cpu().numpy()


@pytest.mark.parametrize("pattern", ["ordinary", "equal", "levels", "outlier", "signed", "rising"])
@pytest.mark.parametrize("lens,k", [((1023, 1, 64), 63), ((1025, 0, 2049), 1024), ((4096,), 1), ((16384,), 16383),
                                    ((16385,), 2048), ((65536,), 700), ((65537,), 33000), ((20000, 900), 9000)])
def test_selection_is_exact(gpu, pattern, lens, k):
    print(f"[case] select {pattern} {lens} k={k}", flush=True)
    rng = np.random.default_rng(17)
    z = scores(pattern, 2, sum(lens), rng)
    _, _, _, cu, got, _, _ = decode(gpu, lens, 2, 1, 64, k, z, rng)
    for b, n in enumerate(lens):
        for h in range(2):
            zs = z[h, cu[b]:cu[b + 1]] + np.float32(0.0)
            want = np.sort(np.argsort(-zs, kind="stable")[: min(k, n)]) + cu[b]
            assert (got[b, h, : min(k, n)] == want).all(), (b, h)


# One sequence far above the average: read again in every pass because the form for shorter ones was chosen (16
# registers: 20001 keys; 64: 66001 keys of 24 heads), or left to the sliced launches (66001 keys of two heads, the
# last time with a window that keeps all of them), with and without the caller's bound.
@pytest.mark.parametrize("pattern", ["ordinary", "equal", "levels", "outlier", "signed", "rising"])
@pytest.mark.parametrize("H_q,lens,k", [(2, (20001, 1, 700, 900), 9000), (24, (66001, 300, 5, 1000), 700),
                                        (2, (300, 66001, 0, 1000), 700), (2, (66001, 5, 900), 67000)])
def test_selection_of_a_skewed_batch(gpu, pattern, H_q, lens, k):
    print(f"[case] select skewed {pattern} {H_q} heads {lens} k={k}", flush=True)
    rng = np.random.default_rng(19)
    z = scores(pattern, H_q, sum(lens), rng)
    lists = []
    for bound in (0, max(lens)):
        _, _, _, cu, got, o, _ = decode(gpu, lens, H_q, 1, 64, k, z, np.random.default_rng(5), max_seqlen=bound)
        lists.append(got)
        assert np.isfinite(o).all()
    for b, n in enumerate(lens):
        for h in range(H_q):
            zs = z[h, cu[b]:cu[b + 1]] + np.float32(0.0)
            want = np.sort(np.argsort(-zs, kind="stable")[: min(k, n)]) + cu[b]
            for got in lists:
                assert (got[b, h, : min(k, n)] == want).all(), (b, h)


@pytest.mark.parametrize("H_q,H_kv,d,lens,k", [(3, 1, 128, (700, 5, 0, 257, 1300), 513), (6, 3, 64, (1030,), 256),
                                               (5, 5, 256, (300, 600, 255), 257), (8, 1, 128, (2000, 1), 1025)])
def test_gather_of_any_group_count(gpu, H_q, H_kv, d, lens, k):
    print(f"[case] gather {H_q}/{H_kv} d={d} {lens}", flush=True)
    rng = np.random.default_rng(23)
    z = scores("ordinary", H_q, sum(lens), rng)
    q, K, V, cu, got, o, lse = decode(gpu, lens, H_q, H_kv, d, k, z, rng, max_seqlen=max(lens))
    ro, rl, rk = orc.dma_decode(q, K, V, z.astype(np.float64), cu, k)
    for b in range(len(lens)):
        assert (got[b, :, : rk[b].shape[1]] == rk[b]).all()
    check_close("o", o, ro, **tol(True))
    fin = np.isfinite(rl)
    assert (np.isneginf(lse) == ~fin).all()
    check_close("lse", lse[fin], rl[fin], **tol(True))


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("bf16", 256), ("f32", 128)])
@pytest.mark.parametrize("lens,k", [((1, 5, 63), 64), ((255, 257, 300), 300), ((700, 2049, 2500), 4096), ((900, 40), 300)])
def test_infinite_value_of_the_last_key(gpu, dtype, d, lens, k):
    """An infinite value in a sequence's newest key gives an infinity where that key is kept, as the sum of
    Eq. 6 does, and nothing where it is not: the rows past the end of a list or of its chunks do not count."""
    print(f"[case] infinite value {dtype} d={d} {lens} k={k}", flush=True)
    T, n_docs, H_q, H_kv = sum(lens), len(lens), 4, 2
    r = np.random.default_rng(29)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = lambda *s: torch.from_numpy(r.standard_normal(s).astype(np.float32)).to(gpu).to(dt)
    q, K, V = dev(n_docs, H_q, d), dev(T, H_kv, d), dev(T, H_kv, d)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    for b in range(n_docs):
        V[int(cu[b + 1]) - 1, 1, 3 + b] = float("inf")
    z = torch.from_numpy(scores("ordinary", H_q, T, r)).to(gpu)
    shape = B.make_shape(T=T, n_docs=n_docs, H_q=H_q, H_kv=H_kv, d=d, k=k, dtype=B.DMA_BF16 if dtype == "bf16" else B.DMA_F32)
    nb, kcap = B.dma_decode_kept_bytes(shape), min(k, T)
    kept = torch.full((nb // 4,), -7, dtype=torch.int32, device=gpu)
    o, lse = torch.zeros((n_docs, H_q, d), dtype=dt, device=gpu), torch.zeros((H_q, n_docs), device=gpu)
    B.dma_decode(shape, q, K, V, z, torch.from_numpy(cu).to(gpu), o, lse, kept, nb)
    lists, out = kept.cpu()[: n_docs * H_q * kcap].view(n_docs, H_q, kcap), o.float().cpu()
    assert torch.isfinite(lse).all() and not torch.isnan(out).any()
    for b, n in enumerate(lens):
        for h in range(H_q):
            want = torch.zeros(d, dtype=torch.bool)
            want[3 + b] = h // 2 == 1 and int(cu[b + 1]) - 1 in lists[b, h, : min(k, n)].tolist()
            assert torch.equal(torch.isposinf(out[b, h]), want), (b, h)
            assert torch.isfinite(out[b, h][~want]).all(), (b, h)
