"""Plans of documents no longer than the window, which are written without a selection, against the general path:
the same shape without the caller's length bound (max_seqlen = 0) selects as usual.  And the same call with a bound
that is too small for some of its documents: no result depends on the bound."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2508_02124_amd import binding as B
from paper_2508_02124_amd import workloads as wlmod
from paper_2508_02124_amd.device_case import DeviceCase
from test_gpu_parity import check_gradients, check_mask

pytestmark = pytest.mark.gpu


def plan(gpu, lens, H_q, H_kv, d, k, max_seqlen, V, W, A):
    T = sum(lens)
    cu = torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int32, device=gpu)
    shape = B.make_shape(T=T, n_docs=len(lens), H_q=H_q, H_kv=H_kv, d=d, k=k, max_seqlen=max_seqlen)
    mask = torch.full((B.dma_mask_bytes(shape),), 0x55, dtype=torch.uint8, device=gpu)
    z = torch.empty((H_q, T), device=gpu)
    expiry = torch.full((H_q, T), -9, dtype=torch.int32, device=gpu)
    topk = torch.full((H_q, T, min(k, T)), -9, dtype=torch.int32, device=gpu)
    if k <= T:
        B.dma_mask_gen(shape, V, W, A, cu, z, expiry, topk, mask)
    else:
        B.dma_mask_gen(shape, V, W, A, cu, z, expiry, None, mask)
    lay = B.dma_mask_describe(shape)
    buf = mask.cpu()

    def view(off, n, *dims):
        return buf[off:off + 4 * n].view(torch.int32).view(*dims)
    nb, kp, mp = lay.nblk_cap, lay.kpad, lay.max_partial
    cnt = view(lay.off_partial_count, H_q * nb, H_q, nb)
    lists = view(lay.off_partial_list, H_q * nb * mp, H_q, nb, mp)
    kept = [lists[h, b, :cnt[h, b]].tolist() for h in range(H_q) for b in range(nb)]
    return z.cpu(), expiry.cpu(), topk.cpu(), cnt, kept, view(lay.off_slot_table, H_q * nb * kp, H_q, nb, kp)


@pytest.mark.parametrize("lens,k", [((1,), 1), ((255, 256, 257), 257), ((0, 5, 0, 600), 600), ((1019,), 1019),
                                    ((513, 512, 1), 1000), ((300, 300), 4096)])
def test_all_kept_plan_equals_the_selected_one(gpu, lens, k):
    print(f"[case] all kept {lens} k={k}", flush=True)
    H_q, H_kv, d, T = 4, 2, 64, sum(lens)
    gen = torch.Generator(device=gpu)
    gen.manual_seed(7)
    V = torch.randn((T, H_kv, d), generator=gen, device=gpu).to(torch.bfloat16)
    W = torch.randn((H_q, d), generator=gen, device=gpu) / 8
    A = -torch.ones(H_q, device=gpu)
    short = plan(gpu, lens, H_q, H_kv, d, k, max(lens), V, W, A)
    # a padding document longer than the window keeps the general path
    longer = lens + (k + 1,)
    V2 = torch.cat([V, torch.randn((k + 1, H_kv, d), generator=gen, device=gpu).to(torch.bfloat16)])
    full = plan(gpu, longer, H_q, H_kv, d, k, 0, V2, W, A)
    nblk = sum((n + 255) // 256 for n in lens)
    assert torch.equal(short[0], full[0][:, :T]) and torch.equal(short[1], full[1][:, :T])
    if k <= T:
        assert torch.equal(short[2], full[2][:, :T])
    assert torch.equal(short[3][:, :nblk], full[3][:, :nblk]) and (short[3][:, nblk:] == 0).all()
    nb_s, nb_f = short[3].shape[1], full[3].shape[1]
    for h in range(H_q):
        for b in range(nblk):
            assert short[4][h * nb_s + b] == full[4][h * nb_f + b]
    kp = min(short[5].shape[2], full[5].shape[2])
    assert torch.equal(short[5][:, :nblk, :kp], full[5][:, :nblk, :kp])


@pytest.mark.parametrize("pattern", ["random", "levels", "rising", "falling"])
@pytest.mark.parametrize("lens,k,bound", [((900, 40, 600), 300, 300), ((257, 1), 256, 200), ((700, 3), 40, 40),
                                          ((30,) * 300 + (70, 513), 64, 64)])
def test_results_do_not_depend_on_the_length_bound(gpu, pattern, lens, k, bound):
    wl = wlmod.small_workload(f"bound_{pattern}_{bound}_below_{max(lens)}", 37, 2, 1, 64, k, lens)
    print(f"[case] {wl.name} k={k}", flush=True)
    inp = wlmod.make_inputs(wl)
    rng = np.random.default_rng(k)
    z = {"random": np.exp(-np.log1p(np.exp(rng.standard_normal((2, inp.T))))),
         "levels": np.round(rng.random((2, inp.T)) * 12) / 12,
         "rising": np.tile(np.linspace(0.1, 1.5, inp.T), (2, 1)),
         "falling": np.tile(np.linspace(1.5, 0.1, inp.T), (2, 1))}[pattern].astype(np.float32)
    case = DeviceCase(inp, gpu, z_override=z, topk=True)
    case.shape.max_seqlen = bound          # (below the longest document; the plan's layout stays the same)
    assert B.dma_mask_bytes(case.shape) == case.mask.numel()
    case.mask_gen()
    check_mask(case, wl.name)
    case.fwd()
    case.bwd()
    check_gradients(case, z.astype(np.float64), "bf16")
