"""GPU parity of the row-major projection past 64 rows (whole lines of W and of
the hidden rows): every row-block count that the 128-wide (three to eight) and
256-wide (three to five) tiles run with, in one M-tile and in several, partial
last blocks, vocabularies off every tile, K from one half line past the
pipeline's depth, odd numbers of half lines; and shapes whose 512-wide tiles
keep the other schedules.  Bound as for any float32 sum of K exact products:
K * 2^-24 * sum |h||w|; and the packed layout, which takes other kernels, gives
the same bits."""

import numpy as np
import pytest
import torch

import paper_2601_21622_amd as sd

from gpu_util import announce, to_np

pytestmark = pytest.mark.gpu

# rows (batch, positions), K, V
CASES = [((13, 5), 32, 40), ((5, 13), 96, 1003), ((19, 5), 64, 257), ((10, 13), 160, 4099), ((32, 5), 288, 20011),
         ((29, 7), 1312, 9001), ((57, 4), 320, 12289), ((51, 5), 96, 33000), ((60, 11), 224, 2049),
         ((64, 5), 544, 32001), ((40, 3), 1504, 30001), ((128, 7), 416, 5000),
         # 128-wide with six blocks; 256-wide with three to five in one M-tile, three and four in two
         ((24, 8), 224, 9001), ((12, 8), 96, 60000), ((32, 4), 160, 50000), ((20, 8), 64, 60001), ((24, 8), 224, 50021),
         ((28, 8), 96, 60000)]


def _row_tile(M, V):
    """Tile width, M-tiles and 32-row blocks per M-tile if the row schedule runs
    (its tile is the one that the deep shapes' price picks), else None."""
    blocks, best = -(-M // 32), None
    for nb, nw, cap in ((1, 4, 12), (2, 4, 7), (2, 8, 5), (4, 4, 7)):
        mt = -(-blocks // cap)
        mb = -(-blocks // mt)
        wgs = -(-V // (32 * nb * nw)) * mt
        cost = -(-wgs // 256) * ((2.1 + mt - 1) / mt * 32 * nb * nw + 32 * mb)
        if best is None or cost < best[0]:
            best = (cost, 32 * nb * nw)
    if best[1] == 512:
        return None
    mt = -(-blocks // {128: 8, 256: 5}[best[1]])
    return best[1], mt, -(-blocks // mt)


def test_cases_cover_every_row_tile():
    ran = [_row_tile(b * g, V) for (b, g), _, V in CASES]
    for ((b, g), K, V), tile in zip(CASES, ran):
        name = sd.sd_vocab_kernel_name(sd.Dims(b, g - 1, 1, 1, 64, K, V, sd.SD_DTYPE_BF16, 0))
        assert (name == "vocab_bf16_rows_kernel") == (tile is not None), (b * g, V, name)
    ran = [t for t in ran if t]
    assert {(t, mb) for t, _, mb in ran} == {(128, n) for n in range(3, 9)} | {(256, n) for n in range(3, 6)}
    assert {(t, mt > 1) for t, mt, _ in ran} == {(t, many) for t in (128, 256) for many in (False, True)}


@pytest.mark.parametrize("rows,K,V", CASES)
def test_row_major_deep_within_rounding_bound(rows, K, V):
    (B, G), M = rows, rows[0] * rows[1]
    announce(f"row schedule M={M} K={K} V={V}")
    g = torch.Generator().manual_seed(M * 1000003 + K * 101 + V)
    h, w = torch.randn(M, K, generator=g).bfloat16(), (torch.randn(V, K, generator=g) / K ** 0.5).bfloat16()
    out = []
    for flags in (0, sd.SD_FLAG_PACKED_VOCAB):
        dims = sd.Dims(B, G - 1, 1, 1, 64, K, V, sd.SD_DTYPE_BF16, flags)
        wd = w.cuda()
        if flags:
            wp = torch.empty(sd.sd_vocab_packed_bytes(dims) // 2, dtype=torch.bfloat16, device="cuda")
            sd.sd_pack_vocab(dims, wd, wp)
            wd = wp
        logits, lse = torch.full((M, V), float("nan"), device="cuda"), torch.full((M,), float("nan"), device="cuda")
        ws = torch.full((sd.sd_workspace_bytes(dims, G),), 0xA5, dtype=torch.uint8, device="cuda")
        sd.sd_verify_logits(dims, h.cuda(), wd, logits, lse, ws)
        out.append((to_np(logits), to_np(lse)))
    hd, wdd = h.double().numpy(), w.double().numpy()
    bound = K * 2.0 ** -24 * (np.abs(hd) @ np.abs(wdd).T) + 1e-30
    assert np.all(np.abs(out[0][0].astype(np.float64) - hd @ wdd.T) <= bound)
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
