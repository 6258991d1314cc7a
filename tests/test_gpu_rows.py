"""GPU parity of the row-major projection past 64 rows (whole lines of W and of
the hidden rows): every row-block count of the 128- and 256-wide tiles with
partial last blocks, several M-tiles, vocabularies off every tile, K from one
half line past the pipeline's depth, odd numbers of half lines.  Bound as for
any float32 sum of K exact products: K * 2^-24 * sum |h||w|; and the packed
layout, which takes other kernels, gives the same bits."""

import numpy as np
import pytest
import torch

import paper_2601_21622_amd as sd

from gpu_util import announce, to_np

pytestmark = pytest.mark.gpu

# rows (batch, positions), K, V
CASES = [((13, 5), 32, 40), ((5, 13), 96, 1003), ((19, 5), 64, 257), ((10, 13), 160, 4099), ((32, 5), 288, 20011),
         ((29, 7), 1312, 9001), ((57, 4), 320, 12289), ((51, 5), 96, 33000), ((60, 11), 224, 2049),
         ((64, 5), 544, 32001), ((40, 3), 1504, 30001), ((128, 7), 416, 5000)]


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
