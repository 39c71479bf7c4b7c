"""GPU parity of single-query attention over ragged caches in both block orders (heads or ranges as the fastest block
index), against the fp64 oracle, sequence by sequence: ranges that end inside a tile, and past a short sequence.  How many
ranges a call was cut into is read off the partial rows that it wrote."""
import math

import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,dh,max_pos,cap,ranges", [
    (12, 8, 8, 128, 1599, 1600, 2),      # heads first
    (3, 8, 8, 128, 999, 1024, 4),
    (2, 32, 2, 128, 900, 960, 4),        # two passes of 8 query heads per cache head
    (4, 16, 16, 128, 1999, 2000, 4),     # 256 blocks, whole rounds over 256 CUs: ranges first
    (5, 16, 16, 128, 1399, 1408, 3),
    (3, 12, 4, 64, 699, 1024, 3),
    (1, 8, 8, 128, 2049, 4096, 9),
    (7, 12, 12, 64, 1799, 1856, 5),
    (21, 12, 12, 64, 800, 832, 1),       # one block per head and sequence, 8 waves
    (40, 12, 12, 64, 800, 832, 1),       # ... 4 waves
])
def test_ragged_decode(B, Hq, Hkv, dh, max_pos, cap, ranges):
    from paper_2604_16498_amd import binding as F
    pos = [int(max_pos * (1 - (i / max(1, B - 1)) ** 2 * 0.97)) for i in range(B)]
    q = I.normal(75, 0, "q", (B, Hq, 1, dh), 1.0, bf16=True)
    k = I.normal(75, 0, "k", (B, Hkv, cap, dh), 1.0, bf16=True)
    v = I.normal(75, 0, "v", (B, Hkv, cap, dh), 1.0, bf16=True)
    ref = np.concatenate([O.attention(q[b:b + 1], k[b:b + 1, :, :n + 1], v[b:b + 1, :, :n + 1], 1.0 / math.sqrt(dh), True)
                          for b, n in enumerate(pos)])
    need = F.forge_attn_fused_workspace_bytes(B, Hq, Hkv, 1, max_pos + 1, dh, torch.bfloat16)
    ws = torch.full((max(need, 4),), 0xff, dtype=torch.uint8, device="cuda")       # NaN patterns that no partial has
    out = torch.empty(B, 1, Hq * dh, dtype=torch.bfloat16, device="cuda")
    F.forge_attn_decode_varlen(dev(q, True), dev(k, True), dev(v, True), out,
                               torch.tensor(pos, dtype=torch.int32, device="cuda"), max_pos, workspace=ws)
    torch.cuda.synchronize()
    check(out, ref, True, "ragged decode")
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        written = int((ws[:ws.numel() // 4 * 4].view(torch.int32) != -1).sum())
        assert written == (B * Hq * ranges * (dh + 2) if ranges > 1 else 0)
