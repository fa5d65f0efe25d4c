"""The pipelined query-stationary kernels at the edges of their tiles: clean tile counts of every remainder of the ring,
documents that end inside a block, each form that the dispatch chooses, and rows whose reference maximum moves again and
again (forward)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle as orc
from paper_2508_02124_amd import workloads as wlmod
from gpu_harness import DeviceCase, check_close, tol
from test_gpu_parity import check_gradients

pytestmark = pytest.mark.gpu

# q-heads, kv-heads, head dimension, documents, windows.  At 128 channels: half blocks with 64-key tiles (few blocks),
# half blocks with 32-key tiles (160 blocks on 256 compute units), whole blocks (256 blocks and a short window).
FORMS = {
    "d128_half64": (2, 1, 128, (700, 33, 515), (1, 31, 33, 64, 65, 129, 193, 256, 300)),
    "d128_half32": (32, 8, 128, (1280,), (33, 100, 200)),
    # (192 blocks: documents that end inside a block, second halves that are partial or empty)
    "d128_half32_ragged": (32, 8, 128, (700, 33, 515), (1, 31, 33, 65, 97, 129)),
    "d128_whole": (32, 8, 128, (1025, 1023), (65, 130, 200)),
    "d256": (2, 1, 256, (700, 33, 515), (1, 31, 33, 64, 65, 97, 129, 300)),
    "d64": (2, 1, 64, (700, 33, 515), (1, 31, 33, 64, 65, 129, 193, 300)),
}


def forward(gpu, name, k, grow):
    H_q, H_kv, d, lens, _ = FORMS[name]
    inp = wlmod.make_inputs(wlmod.small_workload(f"{name}_k{k}", 900 + k, H_q, H_kv, d, k, lens))
    if grow:  # scores that climb along the keys by far more than 2^8 in the weights, with steps up and down on the way
        j = np.arange(inp.T, dtype=np.float32)
        slope = (j / 40 + 8 * np.sin(j / 9)) / np.sqrt(d)
        inp.Q[:] = wlmod.bf16_bits_to_f32(wlmod.f32_to_bf16_bits(0.25 * inp.Q + 1))
        inp.K[:] = wlmod.bf16_bits_to_f32(wlmod.f32_to_bf16_bits(0.25 * inp.K + slope[:, None, None]))
        for x in ("Q", "K"):
            inp.bits[x] = wlmod.f32_to_bf16_bits(getattr(inp, x))
    case = DeviceCase(inp, gpu)
    case.mask_gen()
    case.fwd()
    heads = sorted({0, H_q - 1})
    O, LSE = orc.dma_forward(inp.Q, inp.K, inp.V, case.host("z"), inp.cu_seqlens, k, heads=heads)[:2]
    check_close(f"O {name} k={k}", case.host("O")[:, heads], np.asarray(O)[:, heads], **tol(True))
    check_close(f"LSE {name} k={k}", case.host("LSE")[heads], np.asarray(LSE)[heads], **tol(True))


@pytest.mark.parametrize("grow", [False, True], ids=["plain", "climbing"])
@pytest.mark.parametrize("name", FORMS)
def test_forward_forms(gpu, name, grow):
    for k in FORMS[name][4]:
        print(f"[case] forward {name} k={k} climbing={grow}", flush=True)
        forward(gpu, name, k, grow)


# dq: whole blocks at 128 channels from 129 blocks of 256 rows on, half blocks of 64-key tiles below
GRADIENTS = {
    "d128_half64": (2, 1, 128, (700, 33, 515), (31, 64, 65, 129, 193, 300)),
    # (two q-heads per kv-head: every dS enters dK rounded to bf16, an error of up to 2^-9 sum_i |dS_i q_i| over all rows and
    # heads of the group; with 34 heads in one group the early keys of a window of 65 exceed the plain bound's 2e-2)
    "d128_whole": (34, 17, 128, (700, 33, 255), (65, 129)),
    "d256": (2, 1, 256, (700, 33, 515), (31, 64, 65, 97, 129, 300)),
    "d64": (2, 1, 64, (700, 33, 515), (31, 64, 65, 129, 193, 300)),
}


@pytest.mark.parametrize("name", GRADIENTS)
def test_gradient_forms(gpu, name):
    H_q, H_kv, d, lens, windows = GRADIENTS[name]
    for k in windows:
        print(f"[case] gradients {name} k={k}", flush=True)
        inp = wlmod.make_inputs(wlmod.small_workload(f"{name}_k{k}", 950 + k, H_q, H_kv, d, k, lens))
        case = DeviceCase(inp, gpu)
        case.mask_gen()
        case.fwd()
        case.bwd()
        check_gradients(case, case.host("z").astype(np.float64), "bf16", label=f"{name} k={k} ")


def test_gradients_of_rows_that_are_never_kept(gpu):
    """Enough rows, few enough of them kept, for the conversion that does not read the others: every row is written."""
    print("[case] sparse conversion", flush=True)
    k, lens = 100, (1000,) * 20 + (1,)
    inp = wlmod.make_inputs(wlmod.small_workload("sparse_rows", 990, 4, 2, 128, k, lens))
    case = DeviceCase(inp, gpu)   # (outputs start as NaN)
    case.mask_gen()
    case.fwd()
    case.bwd()
    check_gradients(case, case.host("z").astype(np.float64), "bf16", label="sparse rows ")
    never = (case.host("expiry") == np.arange(inp.T)[None, :]).reshape(2, 2, inp.T).all(axis=1)  # [kv-head, token]
    assert 0.3 < never.mean() < 0.9
    assert (case.host("dK").transpose(1, 0, 2)[never] == 0).all() and (case.host("dV").transpose(1, 0, 2)[never] == 0).all()


# q-heads, kv-heads, head dimension, documents: at least 2^22 elements of dK, and rows that do not fill the last workgroup
SPARSE = {"d64": (4, 4, 64, (1000,) * 17 + (13,)), "d128": (4, 1, 128, (1100,) * 30 + (7,)), "d256": (2, 1, 256, (500,) * 33 + (9,))}


@pytest.mark.parametrize("rising", [False, True], ids=["random", "rising"])
@pytest.mark.parametrize("name", SPARSE)
def test_sparse_conversion_forms(gpu, name, rising):
    """The conversion that leaves out rows, of every head dimension, also where scores that rise along the keys keep all."""
    print(f"[case] sparse conversion {name} rising={rising}", flush=True)
    H_q, H_kv, d, lens = SPARSE[name]
    inp = wlmod.make_inputs(wlmod.small_workload(f"sparse_{name}", 991, H_q, H_kv, d, 48, lens))
    assert inp.T * H_kv * d >= 1 << 22
    z = np.tile(np.linspace(0.1, 1, inp.T, dtype=np.float32), (H_q, 1)) if rising else None
    case = DeviceCase(inp, gpu, z_override=z)
    case.mask_gen()
    case.fwd()
    case.bwd()
    kept = (case.host("expiry") > np.arange(inp.T)[None, :]).reshape(H_kv, H_q // H_kv, inp.T).any(axis=1)
    assert kept.all() if rising else kept.mean() < 0.6
    for out in ("dK", "dV"):
        assert (case.host(out).transpose(1, 0, 2)[~kept] == 0).all()
    check_gradients(case, case.host("z").astype(np.float64), "bf16", label=f"{name} rising={rising} ")


@pytest.mark.parametrize("what", ["V", "K"])
@pytest.mark.parametrize("rising", [False, True], ids=["", "rising"])
@pytest.mark.parametrize("name", FORMS)
def test_an_infinite_entry_stays_with_the_rows_of_its_unit(gpu, name, rising, what):
    """One infinite entry of V or K.  Of the rows that do not keep its key, only those may lose their O or dQ that share a
    step with it: the 32 rows of a wave on which some key of the same 32 entries of the block's list is active.  Rising
    scores and a window of 40: a block's list begins with the last 40 keys of the block, which most waves do not keep."""
    H_q, H_kv, d, lens, windows = FORMS[name]
    k = 40 if rising else windows[-1]
    inp = wlmod.make_inputs(wlmod.small_workload(f"inf_{name}", 970, H_q, H_kv, d, k, lens))
    z = np.tile(np.linspace(0.1, 1, inp.T, dtype=np.float32), (H_q, 1)) if rising else None
    case = DeviceCase(inp, gpu, z_override=z)
    case.mask_gen()
    z, e, pv = case.host("z").copy(), case.host("expiry").copy(), case.plan_views()
    rows = np.arange(inp.T)
    ever = [j for j in range(3, inp.T, 29) if (e[:H_q // H_kv, j] > j).any()][:24]
    assert len(ever) > 8
    for j in ever:
        print(f"[case] {name}: infinite {what} of key {j}", flush=True)
        case = DeviceCase(inp, gpu, z_override=z)
        getattr(case, what)[j, 0, 5] = float("inf")
        case.mask_gen()
        case.fwd()
        case.bwd()
        for h in range(H_q // H_kv):
            lost = (rows >= j) & (rows < e[h, j])
            for b in range(pv["nblk"]):
                r0, r1 = pv["blk"][b][1:3]
                entries = pv["plist"][h, b, :pv["pcnt"][h, b]]
                at = np.flatnonzero(entries == j)
                if at.size:
                    unit = entries[at[0] // 32 * 32:][:32]
                    for r in range(r0, r1, 32):
                        if ((unit <= r + 31) & (e[h, unit] > r)).any():
                            lost[r:min(r + 32, r1)] = True
            for out in ("O", "dQ"):
                bad = ~np.isfinite(case.host(out)[:, h]).all(axis=1)
                assert not (bad & ~lost).any(), (out, h, np.flatnonzero(bad & ~lost)[:8])
        for out in ("O", "dQ"):
            assert np.isfinite(case.host(out)[:, H_q // H_kv:]).all()
