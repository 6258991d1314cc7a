"""GPU parity of the projection's line schedule (float32, and bfloat16 with at
most 64 rows): every pair of a row-block count and a number of waves per
workgroup (chosen from the sizes) in each layout, M-tiles of float32 past 64
rows, rows and vocabularies off every tile, K from one half line (bfloat16: 32
entries) past the pipeline's depth, odd numbers of half lines.

Bound: a float32 sum of K products in any order is within K * 2^-24 * sum
|h||w| of the exact one (products of float32 inputs add one rounding each;
those of bfloat16 are exact)."""

import numpy as np
import pytest
import torch

import paper_2601_21622_amd as sd

from gpu_util import announce

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, rows (batch, positions), K, V, packed
    ("f32", (1, 2), 32, 1, False), ("f32", (3, 5), 64, 33, False), ("f32", (4, 4), 96, 15, False),
    ("f32", (1, 17), 320, 3001, False), ("f32", (8, 6), 544, 12301, False), ("f32", (13, 5), 160, 24700, False),
    ("f32", (26, 5), 288, 129, False), ("f32", (16, 4), 1024, 25000, False),
    ("bf16", (1, 2), 32, 17, False), ("bf16", (1, 2), 32, 17, True), ("bf16", (4, 4), 64, 1, True),
    ("bf16", (1, 17), 96, 3001, False), ("bf16", (1, 17), 96, 3001, True), ("bf16", (8, 6), 352, 12301, False),
    ("bf16", (8, 6), 352, 12301, True), ("bf16", (7, 7), 1312, 24700, False), ("bf16", (7, 7), 1312, 24700, True),
    ("bf16", (16, 4), 1504, 24703, False), ("bf16", (16, 4), 512, 65, True),
    # Rows a multiple of 4 KB apart: the tiles start on different lines.
    ("bf16", (3, 2), 2048, 4001, False), ("bf16", (3, 2), 2048, 4001, True), ("bf16", (8, 6), 4096, 2500, False),
    ("f32", (2, 3), 1024, 3000, False), ("f32", (20, 4), 1024, 700, False),
    # Vocabularies from a few waves' to more than a workgroup per CU.
    *[("bf16", (2, 4), 96, 16 * nw * 250 + 5, nw % 2 == 0) for nw in range(1, 9)],
    *[("f32", (16, 4), 64, 16 * nw * 250 - 3, False) for nw in range(1, 9)],
]


@pytest.mark.parametrize("dtype,rows,K,V,packed", CASES)
def test_line_schedule_within_rounding_bound(dtype, rows, K, V, packed):
    (B, G), M = rows, rows[0] * rows[1]
    announce(f"line schedule dtype={dtype} M={M} K={K} V={V} packed={packed}")
    g = torch.Generator().manual_seed(M * 1000003 + K * 101 + V)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    h, w = torch.randn(M, K, generator=g).to(dt), (torch.randn(V, K, generator=g) / K ** 0.5).to(dt)
    dims = sd.Dims(B, G - 1, 1, 1, 64, K, V, sd.SD_DTYPE_F32 if dtype == "f32" else sd.SD_DTYPE_BF16,
                   sd.SD_FLAG_PACKED_VOCAB if packed else 0)
    wd = w.cuda()
    if packed:
        wp = torch.empty(sd.sd_vocab_packed_bytes(dims) // 2, dtype=dt, device="cuda")
        sd.sd_pack_vocab(dims, wd, wp)
        wd = wp
    logits = torch.full((M, V), float("nan"), device="cuda")
    lse = torch.full((M,), float("nan"), device="cuda")
    ws = torch.full((sd.sd_workspace_bytes(dims, G),), 0xA5, dtype=torch.uint8, device="cuda")
    sd.sd_verify_logits(dims, h.cuda(), wd, logits, lse, ws)
    hd, wdd = h.double().numpy(), w.double().numpy()
    ref = hd @ wdd.T
    bound = K * 2.0 ** -24 * (np.abs(hd) @ np.abs(wdd).T) + 1e-30
    got = logits.cpu().double().numpy()
    assert np.all(np.abs(got - ref) <= bound), float(np.max(np.abs(got - ref) / bound))
    mx = got.max(axis=1, keepdims=True)
    want = (mx + np.log(np.exp(got - mx).sum(axis=1, keepdims=True)))[:, 0]
    # exp and the tile sums in float32, the fold in float64, the result rounded to float32
    assert np.all(np.abs(lse.cpu().double().numpy() - want) <= 1e-5 * np.maximum(1.0, np.abs(want)))


@pytest.mark.parametrize("dtype,rows,K,V", [("f32", (1, 5), 256, 1000), ("bf16", (3, 3), 352, 6025), ("f32", (20, 4), 64, 3000)])
def test_line_schedule_in_the_smallest_workspace(dtype, rows, K, V):
    """Statistics of 64-entry tiles are all the workspace that logits need:
    finer tiles are taken only where the workspace holds theirs.  Both plans
    stay within the rounding bound of the sums; less is refused."""
    (B, G), M = rows, rows[0] * rows[1]
    announce(f"smallest workspace dtype={dtype} M={M} K={K} V={V}")
    g = torch.Generator().manual_seed(M + K + V)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    h, w = torch.randn(M, K, generator=g).to(dt), (torch.randn(V, K, generator=g) / K ** 0.5).to(dt)
    dims = sd.Dims(B, G - 1, 1, 1, 64, K, V, sd.SD_DTYPE_F32 if dtype == "f32" else sd.SD_DTYPE_BF16, 0)
    least = (8 * M * ((V + 63) // 64) + 255) // 256 * 256
    hd, wd = h.cuda(), w.cuda()
    logits = torch.full((M, V), float("nan"), device="cuda")
    lse = torch.full((M,), float("nan"), device="cuda")
    room = torch.full((least + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    sd.sd_verify_logits(dims, hd, wd, logits, lse, room[:least])
    ref = h.double().numpy() @ w.double().numpy().T
    bound = K * 2.0 ** -24 * (np.abs(h.double().numpy()) @ np.abs(w.double().numpy()).T) + 1e-30
    got = logits.cpu().double().numpy()
    assert np.all(np.abs(got - ref) <= bound)
    mx = got.max(axis=1, keepdims=True)
    want = (mx + np.log(np.exp(got - mx).sum(axis=1, keepdims=True)))[:, 0]
    assert np.all(np.abs(lse.cpu().double().numpy() - want) <= 1e-5 * np.maximum(1.0, np.abs(want)))
    assert bool((room[least:] == 0xA5).all())
    with pytest.raises(sd.SdError):
        sd.sd_verify_logits(dims, hd, wd, logits, lse, room[:least - 256])


def _waves(M, V):
    """Waves per workgroup and 16-row blocks per M-tile, by the library's price."""
    blocks = -(-M // 16)
    mt = -(-blocks // 4)
    mb = -(-blocks // mt)
    best = None
    for nw in range(8, 0, -1):
        groups = -(-V // (16 * nw)) * mt
        cost = -(-groups // 256) * (16 * nw + 16 * mb + 16) + 1.5 * 16 * mb * groups / 256
        if best is None or cost < best[0]:
            best = (cost, nw)
    return best[1], mb


# A vocabulary that takes each number of waves, per row-block count.
PAIRS = {1: (501, 4201, 8301, 12401, 16501, 20501, 24701, 28801), 2: (501, 2901, 8301, 12401, 16501, 20501, 24701, 28801),
         3: (501, 1901, 5501, 11001, 16501, 20501, 24701, 28801), 4: (501, 1401, 4201, 8301, 13801, 20501, 24701, 28801)}


@pytest.mark.parametrize("mb", sorted(PAIRS))
@pytest.mark.parametrize("kind", ["f32", "bf16", "bf16_packed"])
def test_every_row_block_and_wave_count(kind, mb):
    """K of one half line, of two lines, and of an odd number of half lines past
    the deepest pipeline (eight lines); a partial last row block."""
    dt, packed = (torch.float32 if kind == "f32" else torch.bfloat16), kind == "bf16_packed"
    B, G = (8 * mb - 1, 2)
    M = B * G
    for nw, V in enumerate(PAIRS[mb], 1):
        assert _waves(M, V) == (nw, mb)
        for K in (32, 128, 608):
            announce(f"line schedule {kind} waves={nw} blocks={mb} K={K} V={V}")
            g = torch.Generator(device="cuda").manual_seed(M * 1009 + K * 101 + V)
            h = torch.randn(M, K, generator=g, device="cuda").to(dt)
            w = (torch.randn(V, K, generator=g, device="cuda") / K ** 0.5).to(dt)
            dims = sd.Dims(B, G - 1, 1, 1, 64, K, V, sd.SD_DTYPE_F32 if kind == "f32" else sd.SD_DTYPE_BF16,
                           sd.SD_FLAG_PACKED_VOCAB if packed else 0)
            wd = w
            if packed:
                wd = torch.empty(sd.sd_vocab_packed_bytes(dims) // 2, dtype=dt, device="cuda")
                sd.sd_pack_vocab(dims, w, wd)
            logits = torch.full((M, V), float("nan"), device="cuda")
            lse = torch.full((M,), float("nan"), device="cuda")
            ws = torch.full((sd.sd_workspace_bytes(dims, G),), 0xA5, dtype=torch.uint8, device="cuda")
            sd.sd_verify_logits(dims, h, wd, logits, lse, ws)
            wt = w.double().t().contiguous()
            bound = K * 2.0 ** -24 * (h.double().abs() @ wt.abs()) + 1e-30
            assert bool(((logits.double() - h.double() @ wt).abs() <= bound).all())
            want = torch.logsumexp(logits.double(), 1)
            assert bool(((lse.double() - want).abs() <= 1e-5 * want.abs().clamp(min=1.0)).all())
