"""Prompt attention on blocks of 2, 4 and 8 waves: the edges of their query blocks (64, 128, 256), key shares on 4 and
8 waves, and the order of the blocks under a mask that all heads share."""
import math

import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


def _qkv(B, Hq, Hkv, Sq, Skv, dh):
    return (I.normal(78, 0, "q", (B, Hq, Sq, dh), 1.0, bf16=True),
            *(I.normal(78, 0, n, (B, Hkv, Skv, dh), 1.0, bf16=True) for n in ("k", "v")))


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Skv,dh", [
    # 2 waves: one block of 64 queries per CU at most
    (1, 4, 2, 2, 2, 64), (1, 4, 4, 63, 63, 128), (1, 2, 2, 64, 191, 64), (2, 3, 1, 65, 65, 128),
    # 4 waves (more than 256 blocks of 64 queries)
    (3, 48, 48, 127, 127, 64), (4, 40, 8, 129, 129, 64), (4, 34, 34, 128, 200, 128), (2, 50, 10, 193, 193, 128),
    # ... in rounds there and back, a broken third one
    (3, 29, 29, 800, 850, 64), (1, 74, 37, 801, 801, 64),
    # 4 waves with shares: the last share short, heads of both sizes
    (1, 4, 4, 33, 1100, 64), (1, 6, 2, 130, 1500, 128),
    # 8 waves: shares, of nine tenths of the chip and of less (the edge in keys too), then whole query blocks well past one round
    (1, 64, 16, 480, 2600, 128), (1, 32, 8, 512, 1700, 128), (2, 16, 4, 750, 1953, 128), (4, 95, 19, 250, 250, 128),
    # ... blocks of even length in less than one round of 8 waves, more than one per CU of 4
    (5, 32, 8, 134, 804, 128),
])
def test_query_blocks(B, Hq, Hkv, Sq, Skv, dh):
    from paper_2604_16498_amd import binding as F
    q, k, v = _qkv(B, Hq, Hkv, Sq, Skv, dh)
    tq, tk, tv = (dev(a, True) for a in (q, k, v))
    out = torch.full((B, Sq, Hq * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = F.workspace(F.forge_attn_fused_workspace_bytes(B, Hq, Hkv, Sq, Skv, dh, torch.bfloat16))
    F.forge_attn_fused(tq, tk, tv, out, workspace=ws)
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
    # the oracle on a handful of heads: the first, the last and two between
    o = out.view(B, Sq, Hq, dh)
    for b, h in {(0, 0), (B - 1, Hq - 1), (B // 2, Hq // 3), (0, Hq - 1)}:
        g = h // (Hq // Hkv)
        ref = O.attention(q[b:b + 1, h:h + 1], k[b:b + 1, g:g + 1], v[b:b + 1, g:g + 1], 1.0 / math.sqrt(dh), True, None)
        check(o[b:b + 1, :, h].contiguous(), ref, True, "head %d of sequence %d" % (h, b))


@pytest.mark.parametrize("per_head", [False, True])
@pytest.mark.parametrize("B,H,S,dh", [(1, 5, 70, 64), (3, 7, 65, 128), (5, 31, 130, 64), (3, 37, 129, 128), (5, 61, 37, 128)])
def test_masked_block_order(B, H, S, dh, per_head):
    """Block counts that are no multiple of 8, a mask of its own per sequence (and per head)."""
    from paper_2604_16498_amd import binding as F
    q, k, v = _qkv(B, H, H, S, S, dh)
    mask = I.normal(78, 0, "misc", (B, H if per_head else 1, S, S), 2.0)
    for b in range(B):
        mask[b, :, :, S - 3 - b:] = -np.inf
    out = torch.full((B, S, H * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    F.forge_attn_fused_masked(*(dev(a, True) for a in (q, k, v)), torch.from_numpy(mask).cuda(), out, causal=False)
    torch.cuda.synchronize()
    check(out, O.attention(q, k, v, 1.0 / math.sqrt(dh), False, mask), True, "masked attention")
