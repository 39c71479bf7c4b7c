"""Decode attention that takes the sequences by length: more blocks than compute units, whole and broken rounds, equal and repeated
lengths, clamped positions, short caches, one range and several in both block orders, up to 64 sequences and more."""
import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from util import check, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,dh,cap", [
    (17, 16, 16, 128, 600), (64, 8, 8, 128, 520),          # a broken second round; two whole ones
    (22, 12, 12, 64, 1030), (65, 8, 8, 64, 1030),          # narrow heads; one sequence too many for a lane each
    (33, 16, 8, 128, 1100), (49, 64, 16, 128, 1030),       # shared heads; more rounds than are resident
    (20, 16, 16, 128, 17), (40, 32, 32, 128, 95), (33, 8, 8, 128, 256), (33, 8, 8, 128, 257),   # short caches in many blocks
])
@pytest.mark.parametrize("lengths", ["spread", "equal", "repeated", "clamped"])
def test_sequences_by_length(B, Hq, Hkv, dh, cap, lengths):
    from paper_2604_16498_amd import binding as F
    rng = np.random.default_rng(B * cap + dh)
    pos = {"spread": rng.integers(0, cap, B), "equal": np.full(B, cap - 3), "repeated": rng.choice([0, 15, cap // 2, cap - 1], B),
           "clamped": rng.choice([-5, 7, cap + 100], B)}[lengths]
    g = torch.Generator(device="cuda").manual_seed(B)
    q, k, v = (torch.randn(B, h, n, dh, generator=g, device="cuda", dtype=torch.bfloat16) for h, n in ((Hq, 1), (Hkv, cap), (Hkv, cap)))
    out = torch.full((B, 1, Hq * dh), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = F.workspace(max(16, F.forge_attn_fused_workspace_bytes(B, Hq, Hkv, 1, cap, dh, torch.bfloat16)))
    F.forge_attn_decode_varlen(q, k, v, out, torch.tensor(pos, dtype=torch.int32, device="cuda"), cap - 1, workspace=ws)
    torch.cuda.synchronize()
    for b in range(B):
        n = int(np.clip(pos[b], 0, cap - 1)) + 1
        ref = O.attention(*(host(t) for t in (q[b:b + 1], k[b:b + 1, :, :n], v[b:b + 1, :, :n])), dh ** -0.5, True)
        check(out[b:b + 1], ref, True, "sequence %d of %d, %d rows" % (b, B, n))


@pytest.mark.parametrize("B,Hq,Hkv,dh,cap,ranges", [
    (17, 8, 8, 128, 1276, 2), (17, 32, 8, 128, 1276, 2),   # heads first, 272 blocks: a broken second round
    (22, 12, 12, 64, 1484, 2), (9, 32, 32, 128, 2040, 2),  # ... a broken third round
    (24, 16, 16, 128, 1400, 2),                            # three whole rounds, ranges first
    (17, 8, 8, 128, 1942, 4), (11, 8, 8, 128, 1054, 3),    # more ranges, heads first and ranges first
    (15, 12, 12, 64, 4200, 3), (8, 12, 12, 64, 1804, 5),   # ... of narrow heads, which stay in batch order
])
@pytest.mark.parametrize("lengths", ["spread", "equal", "repeated", "clamped"])
def test_ranges_by_length(B, Hq, Hkv, dh, cap, ranges, lengths):
    """How many ranges a call was cut into is read off the partial rows that it wrote."""
    from paper_2604_16498_amd import binding as F
    rng = np.random.default_rng(B * cap + dh + 1)
    pos = {"spread": rng.integers(0, cap, B), "equal": np.full(B, cap - 3), "repeated": rng.choice([0, 15, cap // 2, cap - 1], B),
           "clamped": rng.choice([-5, 7, cap + 100], B)}[lengths]
    g = torch.Generator(device="cuda").manual_seed(B)
    q, k, v = (torch.randn(B, h, n, dh, generator=g, device="cuda", dtype=torch.bfloat16) for h, n in ((Hq, 1), (Hkv, cap), (Hkv, cap)))
    out = torch.full((B, 1, Hq * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
    need = F.forge_attn_fused_workspace_bytes(B, Hq, Hkv, 1, cap, dh, torch.bfloat16)
    ws = torch.full((need,), 0xff, dtype=torch.uint8, device="cuda")           # NaN patterns that no partial has
    F.forge_attn_decode_varlen(q, k, v, out, torch.tensor(pos, dtype=torch.int32, device="cuda"), cap - 1, workspace=ws)
    torch.cuda.synchronize()
    for b in range(B):
        n = int(np.clip(pos[b], 0, cap - 1)) + 1
        ref = O.attention(*(host(t) for t in (q[b:b + 1], k[b:b + 1, :, :n], v[b:b + 1, :, :n])), dh ** -0.5, True)
        check(out[b:b + 1], ref, True, "sequence %d of %d, %d rows" % (b, B, n))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert int((ws[:need // 4 * 4].view(torch.int32) != -1).sum()) == B * Hq * ranges * (dh + 2)
