"""GPU parity of the float32 attention at the edges of its tiles: 16-key blocks,
32 keys per wave, 128-key chunks (several per request), one to four 16-row
blocks with remainders, grouped heads, both head dimensions, chain and tree.

Bound: with eps = 2^-24, a score sums D products (error at most D eps sum|q||k|
scale), so a weight is off by at most twice that plus a few eps, relatively,
and so is its normaliser; the output adds L products of weights that sum to
one."""

import math

import numpy as np
import pytest
import torch

import paper_2601_21622_amd as sd
from oracle import tree_attention, verify_attention

from gpu_util import announce, tensor

pytestmark = pytest.mark.gpu

CASES = [
    # D, Hkv, group, G, lengths
    (64, 1, 1, 2, (2, 15, 16, 17, 31, 32, 33)), (64, 2, 3, 5, (5, 127, 128, 129, 300)),
    (128, 2, 1, 16, (16, 64, 95, 97)), (128, 1, 4, 5, (33, 128, 257)), (128, 1, 8, 8, (40, 130)),
    (64, 3, 1, 64, (64, 160)),
]


@pytest.mark.parametrize("tree", [False, True])
@pytest.mark.parametrize("D,Hkv,group,G,lengths", CASES)
def test_f32_attention_within_rounding_bound(D, Hkv, group, G, lengths, tree):
    B, Hq = len(lengths), Hkv * group
    announce(f"f32 attention D={D} Hkv={Hkv} group={group} G={G} lengths={lengths} tree={tree}")
    rng = np.random.default_rng(D * 1000 + G * 10 + group)
    kv_len = np.array(lengths, dtype=np.int32)
    seg = Hkv * kv_len.astype(np.int64) * D
    kv_off = np.concatenate([[0], np.cumsum(seg)[:-1]]).astype(np.int64)
    q = rng.standard_normal((B, G, Hq, D)).astype(np.float32)
    k, v = (rng.standard_normal(int(seg.sum())).astype(np.float32) for _ in range(2))
    dims = sd.Dims(B, G - 1, Hq, Hkv, D, 32, 64, sd.SD_DTYPE_F32, 0)
    out = torch.full((B, G, Hq, D), float("nan"), device="cuda")
    ws = torch.full((sd.sd_workspace_bytes(dims, int(kv_len.max())),), 0xA5, dtype=torch.uint8, device="cuda")
    scale = 1.0 / math.sqrt(D)
    if tree:
        parent = np.stack([[int(rng.integers(-1, i)) for i in range(G - 1)] for _ in range(B)]).astype(np.int32)
        sd.sd_verify_attention_tree(dims, tensor(q), tensor(k), tensor(v), kv_off, kv_len, tensor(parent), scale, out, ws)
        ref = tree_attention(q, k, v, kv_off, kv_len, Hkv, parent)
    else:
        sd.sd_verify_attention(dims, tensor(q), tensor(k), tensor(v), kv_off, kv_len, scale, out, ws)
        ref = verify_attention(q, k, v, kv_off, kv_len, Hkv)
    eps = 2.0 ** -24
    s_abs = scale * float(np.abs(q).sum(axis=-1).max()) * float(np.abs(k).max())  # bounds sum|q||k| scale
    weight = 2 * (D + 4) * eps * s_abs + 8 * eps
    bound = (2 * weight + (int(kv_len.max()) + 16) * eps) * float(np.abs(v).max())
    assert float(np.max(np.abs(out.cpu().double().numpy() - ref))) <= bound
