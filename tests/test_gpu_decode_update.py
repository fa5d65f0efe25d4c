"""The kept set carried from one decode step to the next, against the best keys of every prefix: lists in registers (up to
2048 keys) and longer ones, the first and the last entry dropped, ties, new keys that do not enter."""
import numpy as np
import pytest
import torch

from paper_2508_02124_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["random", "ties", "rising", "falling"])
@pytest.mark.parametrize("k", [1, 300, 2048, 2049, 2500])
def test_update(k, kind):
    print(f"[case] update k={k} {kind}", flush=True)
    dev, caps, H, steps = torch.device("cuda"), (3100, 2600, k + 2), 2, 6
    T, cu = sum(caps), np.concatenate([[0], np.cumsum(caps)])
    rng = np.random.default_rng(k)
    z = rng.uniform(0.1, 1, (H, T)).astype(np.float32)
    if kind == "ties":
        z = (np.round(z * 4) / 4).astype(np.float32)
    elif kind != "random":
        z[:] = np.linspace(0.1, 1, T)[::1 if kind == "rising" else -1]
    shape = B.make_shape(T, len(caps), H, 1, 64, k, dtype=B.DMA_BF16)
    K = torch.zeros((T, 1, 64), dtype=torch.bfloat16, device=dev)
    q = torch.zeros((len(caps), H, 64), dtype=torch.bfloat16, device=dev)
    o, lse = torch.empty_like(q), torch.empty((H, len(caps)), device=dev)
    nbytes = B.dma_decode_kept_bytes(shape)
    kept = torch.zeros((nbytes + 3) // 4, dtype=torch.int32, device=dev)
    zt, cut = torch.from_numpy(z).to(dev), torch.from_numpy(cu.astype(np.int32)).to(dev)
    for i in range(steps + 1):
        lens = [max(0, c - steps + i) for c in caps]
        B.dma_decode_step(shape, q, K, K, zt, cut, torch.tensor(lens, dtype=torch.int32, device=dev), i == 0, o, lse, kept,
                          nbytes)
        lists = kept[: len(caps) * H * k].cpu().numpy().reshape(len(caps), H, k)
        for b, n in enumerate(lens):
            for h in range(H):
                prefix = z[h, cu[b]:cu[b] + n]
                best = np.sort(np.argsort(-prefix, kind="stable")[:k]) + cu[b]
                assert (lists[b, h, :len(best)] == best).all(), (i, b, h)
