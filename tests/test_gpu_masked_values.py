"""Masked attention whose first key tiles, or whole rows, are cut by large finite values: every block size of the prompt kernel,
single queries, fp32.  The mask may hold any finite value; a row cut throughout by one value is the mean of V where its scores vanish beside it."""
import math

import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import binding as F
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cut", [-1e4, -1e9, -1e10, -1e18, -1e20, -1e29, -2e30, float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("B,H,S,Skv,dh", [
    (2, 3, 130, 193, 64), (4, 20, 260, 300, 64), (9, 58, 97, 200, 64),      # blocks of 2 and of 4 waves, more than two of these per CU
    (2, 3, 130, 193, 128), (5, 54, 97, 200, 128),                           # blocks of 4 and of 8 waves
])
def test_rows_cut_by_large_values(B, H, S, Skv, dh, cut):
    q, k, v = (I.normal(81, 0, n, (B, H, s, dh), 1.0, bf16=True) for n, s in (("q", S), ("k", Skv), ("v", Skv)))
    mask = I.normal(81, 0, "misc", (B, 1, S, Skv), 2.0)
    for i in range(0, S, 3):
        mask[:, :, i, :64 + 13 * (i % 5)] = cut              # left padding, the first tile and more
    vanish = abs(cut) >= 1e9                                 # half an ulp of it is at least 32, more than any score here
    through = np.arange(1, S, 3) if vanish else np.arange(0)
    mask[:, :, through, :] = cut
    out = torch.full((B, S, H * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    F.forge_attn_fused_masked(*(dev(a, True) for a in (q, k, v)), torch.from_numpy(mask).cuda(), out, causal=False)
    torch.cuda.synchronize()
    o = out.view(B, S, H, dh)
    for b, h in {(0, 0), (B - 1, H - 1), (B // 2, H // 2)}:
        ref = O.attention(q[b:b + 1, h:h + 1], k[b:b + 1, h:h + 1], v[b:b + 1, h:h + 1], 1.0 / math.sqrt(dh), False, mask[b:b + 1])
        ref = ref.reshape(S, dh).copy()
        ref[through] = v[b, h].astype(np.float64).mean(0)
        check(o[b, :, h].contiguous(), ref, True, "head %d of sequence %d" % (h, b))


@pytest.mark.parametrize("cut", [-1e9, -1e10, -1e29, -2e30, float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("bf16,S,dh", [(True, 1, 64), (True, 1, 128), (False, 1, 64), (False, 20, 128)])
def test_rows_on_the_vector_alu(bf16, S, dh, cut):
    B, H, Skv = 2, 3, 193
    q, k, v = (I.normal(82, 0, n, (B, H, s, dh), 1.0, bf16=bf16) for n, s in (("q", S), ("k", Skv), ("v", Skv)))
    mask = I.normal(82, 0, "misc", (B, H, S, Skv), 2.0)
    mask[:, 0] = cut                                         # a head cut throughout, one by left padding
    mask[:, 1, :, :70] = cut
    out = torch.full((B, S, H * dh), float("nan"), dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
    F.forge_attn_fused_masked(*(dev(a, bf16) for a in (q, k, v)), torch.from_numpy(mask).cuda(), out, causal=False)
    torch.cuda.synchronize()
    ref = O.attention(q, k, v, 1.0 / math.sqrt(dh), False, mask).reshape(B, S, H, dh).copy()
    ref[:, :, 0] = v[:, 0].astype(np.float64).mean(1)[:, None]
    check(out.view(B, S, H, dh), ref, bf16, "cut by %g" % cut)
