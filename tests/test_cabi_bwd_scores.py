"""dma_bwd_scores refuses what dma_bwd and dma_mask_bwd refuse, before any launch (no GPU needed)."""
import pytest

from paper_2508_02124_amd import binding as B
from test_cabi import lib  # noqa: F401  (the fixture)

P = 0x1000  # aligned dummy address: never dereferenced on a failing call
ARGS = dict(Q=P, K=P, V=P, O=P, dO=P, LSE=P, z=P, expiry=P, mask=P, cu_seqlens=P, W=P, A=P, dQ=P, dK=P, dV=P, dz=P, dW=P,
            dA=P, ws=P, ws_bytes=1 << 40)


@pytest.mark.parametrize("shape,change,status", [
    ({}, dict(W=None), B.DMA_EINVAL), ({}, dict(dA=None), B.DMA_EINVAL), ({}, dict(dQ=None), B.DMA_EINVAL),
    ({}, dict(dW=P + 4), B.DMA_EINVAL), ({}, dict(dz=P + 8), B.DMA_EINVAL), ({}, dict(ws_bytes=16), B.DMA_EWORKSPACE),
    ({"d": 80}, {}, B.DMA_EUNSUPPORTED), ({"H_q": 64, "H_kv": 1, "d": 128}, {}, B.DMA_EUNSUPPORTED)])
def test_refused(lib, shape, change, status):  # noqa: F811
    s = B.make_shape(**{**dict(T=256, n_docs=1, H_q=2, H_kv=2, d=64, k=64), **shape})
    with pytest.raises(B.DmaError) as e:
        B.dma_bwd_scores(s, **{**ARGS, **change}, stream=0)
    assert e.value.status == status
