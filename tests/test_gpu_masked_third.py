"""Masked attention on three blocks per CU (head_dim 64, more than two blocks of 128 queries per CU): ragged ends of queries and keys,
additive values, the last keys cut by -inf, by the type's lowest value and by -1e4, a mask for all heads and one each; causal calls."""
import math

import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import binding as F
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cut", [-np.inf, float(np.finfo(np.float32).min), -1e4])
@pytest.mark.parametrize("B,H,Hkv,S,Skv,per_head", [(9, 58, 58, 97, 97, False), (5, 54, 18, 130, 193, True), (3, 60, 60, 257, 320, False)])
def test_masked_three_blocks(B, H, Hkv, S, Skv, per_head, cut):
    q, k, v = (I.normal(79, 0, n, (B, h, s, 64), 1.0, bf16=True) for n, h, s in (("q", H, S), ("k", Hkv, Skv), ("v", Hkv, Skv)))
    mask = I.normal(79, 0, "misc", (B, H if per_head else 1, S, Skv), 2.0)
    for b in range(B):
        mask[b, :, :, Skv - 65 - b:] = cut
    out = torch.full((B, S, H * 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    F.forge_attn_fused_masked(*(dev(a, True) for a in (q, k, v)), torch.from_numpy(mask).cuda(), out, causal=False)
    torch.cuda.synchronize()
    o = out.view(B, S, H, 64)
    for b, h in {(0, 0), (B - 1, H - 1), (B // 2, H // 3), (1, 7)}:
        g = h // (H // Hkv)
        m = mask[b:b + 1, h:h + 1] if per_head else mask[b:b + 1]
        ref = O.attention(q[b:b + 1, h:h + 1], k[b:b + 1, g:g + 1], v[b:b + 1, g:g + 1], 1.0 / math.sqrt(64), False, m)
        check(o[b:b + 1, :, h].contiguous(), ref, True, "head %d of sequence %d" % (h, b))


@pytest.mark.parametrize("B,H,S,Skv,per_head", [
    (9, 58, 97, 97, False), (3, 60, 257, 320, True),     # a third block per CU
    (3, 29, 800, 850, False), (1, 77, 800, 801, True),   # seven query blocks per head, 609 and 539 blocks: the second round backwards
])
def test_masked_causal_many_blocks(B, H, S, Skv, per_head):
    """Tiles that a wave skips, and rows of query blocks that cross a round of the chip, under one mask for all heads and one each."""
    q, k, v = (I.normal(80, 0, n, (B, H, s, 64), 1.0, bf16=True) for n, s in (("q", S), ("k", Skv), ("v", Skv)))
    mask = np.repeat(I.normal(80, 0, "misc", (B, H if per_head else 1, 1, Skv), 2.0), S, axis=2)
    mask[:, :, 5::7, 1:70] = -np.inf
    out = torch.full((B, S, H * 64), float("nan"), dtype=torch.bfloat16, device="cuda")
    F.forge_attn_fused_masked(*(dev(a, True) for a in (q, k, v)), torch.from_numpy(mask).cuda(), out, causal=True)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    o = out.view(B, S, H, 64)
    for b, h in {(0, 0), (B - 1, H - 1), (B // 2, H // 3), (0, H - 2)}:
        m = mask[b:b + 1, h:h + 1] if per_head else mask[b:b + 1]
        ref = O.attention(q[b:b + 1, h:h + 1], k[b:b + 1, h:h + 1], v[b:b + 1, h:h + 1], 0.125, True, m)
        check(o[b:b + 1, :, h].contiguous(), ref, True, "head %d of sequence %d" % (h, b))
