"""The causal selection by blocks (select.hip) against the sequential oracle: expiries of every key, bit for bit, at block,
window and checkpoint edges, for scores whose bins separate them and for scores where they do not (ties, outliers,
infinities, not-a-numbers)."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2508_02124_amd import binding as B

pytestmark = pytest.mark.gpu


def rank_order(z):
    """The order of the scores as the library ranks them: by bits, -0 as +0, a positive NaN above and a negative one below
    everything else; as float64 numbers without infinities."""
    with np.errstate(invalid="ignore"):  # (a signalling NaN becomes a quiet one, here and there)
        u = (z + np.float32(0)).view(np.uint32)
    key = np.where(u >> 31, ~u, u | np.uint32(0x80000000))
    return key.astype(np.float64)


def scores(kind, H, n, rng):
    z = np.exp(-rng.uniform(0.5, 2, (H, 1)) * np.log1p(np.exp(rng.standard_normal((H, n))))).astype(np.float32)
    if kind == "ties":
        z = (np.round(z * 4) / 4).astype(np.float32)
    elif kind == "equal":
        z[:] = 0.5
    elif kind == "rising":
        z[:] = np.linspace(0.1, 1, n, dtype=np.float32)
    elif kind == "falling":
        z[:] = np.linspace(1, 0.1, n, dtype=np.float32)
    elif kind == "outliers":  # one bin holds nearly everything
        z[:, rng.integers(0, n, 3)] = 1e30
        z[:, rng.integers(0, n, 3)] = -1e30
    elif kind == "climbing":  # positive gates: scores over many powers of two, with a zero
        z = np.exp(rng.uniform(2, 6, (H, 1)) * np.log1p(np.exp(2 * rng.standard_normal((H, n))))).astype(np.float32)
        z[:, n // 3] = 0
    elif kind == "signed":
        z = rng.standard_normal((H, n)).astype(np.float32)
    elif kind == "runs":  # few values, each in long runs: the ranks fall among equal keys
        z = (rng.integers(0, 3, (H, n)) / 4).astype(np.float32)
        z[:, n // 5:n // 2] = 0.5
    elif kind == "special":  # infinities, zeros of both signs, subnormals, NaNs of both signs
        pick = rng.integers(0, 12, z.shape)
        special = np.array([np.inf, -np.inf, 0.0, -0.0, 1e-40, -1e-40], dtype=np.float32)
        z = np.where(pick < 6, special[np.minimum(pick, 5)], z).astype(np.float32)
        z[:, n // 3] = np.nan
        z[:, n // 4] = np.array([0x7F800001], dtype=np.uint32).view(np.float32)[0]
        z[:, n // 2] = np.array([0xFFC00000], dtype=np.uint32).view(np.float32)[0]
    return z


def expiries(z, lens, k, max_seqlen):
    H, T = z.shape
    dev = torch.device("cuda")
    shape = B.make_shape(T, len(lens), H, 1, 64, k, dtype=B.DMA_BF16, max_seqlen=max_seqlen)
    V = torch.zeros((T, 1, 64), dtype=torch.bfloat16, device=dev)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=dev)
    zt = torch.from_numpy(z).to(dev)
    e = torch.full((H, T), -7, dtype=torch.int32, device=dev)
    mask = torch.empty(B.dma_mask_bytes(shape), dtype=torch.uint8, device=dev)
    B.dma_mask_gen(shape, V, None, None, cu, zt, e, None, mask)
    return e.cpu().numpy()


def check(z, lens, k, max_seqlen=None):
    got = expiries(z, lens, k, max(lens) if max_seqlen is None else max_seqlen)
    for h in range(z.shape[0]):
        a = 0
        for n in lens:
            if n:
                ref = orc.expiry_sequential(rank_order(z[h, a:a + n]), k) + a
                bad = np.flatnonzero(got[h, a:a + n] != ref)
                assert bad.size == 0, f"head {h}, document at {a}: {bad.size} of {n} differ, first {bad[:5]}"
            a += n


KINDS = ["random", "ties", "equal", "rising", "falling", "outliers", "special", "climbing", "signed", "runs"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("lens,k", [((255, 256, 257, 0, 1), 64), ((700, 513, 300), 300), ((2049, 100), 1), ((1500,), 1023),
                                    ((8192, 8300), 700), ((9000, 5000), 2048)])
def test_expiries(kind, lens, k):
    rng = np.random.default_rng(100 + k)
    check(scores(kind, 2, sum(lens), rng), lens, k)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("lens,k", [((16385, 300), 333), ((20600, 16384), 4096), ((18000,), 9000), ((16600,), 4094), ((17000,), 4097),
                                    ((65536,), 1500)])
def test_expiries_of_long_documents(kind, lens, k):
    rng = np.random.default_rng(200 + k)
    check(scores(kind, 1, sum(lens), rng), lens, k)


@pytest.mark.parametrize("n", [131072, 131073])  # the longest document worked out by blocks; a sorted one
def test_expiries_of_the_longest_documents(n):
    check(scores("random", 1, n, np.random.default_rng(9)), (n,), 1500)


@pytest.mark.parametrize("bound", [0, 500, 17000])
def test_no_expiry_depends_on_the_bound(bound):
    lens, k = (20000, 300, 600), 400
    check(scores("random", 2, sum(lens), np.random.default_rng(7)), lens, k, bound)
