"""GPU parity of the prompt attention whose keys are shared out over several blocks (few query blocks, many
keys), against the fp64 oracle, at shares with remainders and early query blocks whose later shares are
empty."""
import math

import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2604_16498_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("B,Hq,Hkv,Sq,Skv,dh,causal", [
    (1, 4, 2, 2, 2049, 128, True),       # 33 tiles, the last of one key, in eight shares
    (1, 4, 1, 33, 1030, 64, True),
    (1, 3, 3, 700, 1500, 64, True),      # the first query block ends well before the last
    (1, 4, 4, 1500, 1500, 128, True),    # ... and needs fewer tiles than there are shares
    (2, 2, 1, 257, 3001, 128, False),
])
def test_shares_match_the_definition(F, B, Hq, Hkv, Sq, Skv, dh, causal):
    q = I.normal(73, 0, "q", (B, Hq, Sq, dh), 1.0, bf16=True)
    k = I.normal(73, 0, "k", (B, Hkv, Skv, dh), 1.0, bf16=True)
    v = I.normal(73, 0, "v", (B, Hkv, Skv, dh), 1.0, bf16=True)
    ref = O.attention(q, k, v, 1.0 / math.sqrt(dh), causal)
    need = F.forge_attn_fused_workspace_bytes(B, Hq, Hkv, Sq, Skv, dh, torch.bfloat16)
    assert need >= 2 * B * Hq * Sq * (dh + 2) * 4
    sizes = [F.forge_attn_fused_workspace_bytes(B, Hq, Hkv, Sq, n, dh, torch.bfloat16) for n in range(Sq, Skv + 1)]
    assert sizes == sorted(sizes)                            # a buffer for the longer cache serves the shorter
    tq, tk, tv = dev(q, True), dev(k, True), dev(v, True)
    outs = []
    for ws in (F.workspace(need), F.workspace(need), None, F.workspace(need - 256)):     # the last two run unsplit
        out = torch.empty(B, Sq, Hq * dh, dtype=torch.bfloat16, device="cuda")
        F.forge_attn_fused(tq, tk, tv, out, causal=causal, workspace=ws)
        outs.append(out)
    torch.cuda.synchronize()
    check(outs[0], ref, True, "shared keys")
    check(outs[2], ref, True, "unsplit")
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[2], outs[3])


@pytest.mark.parametrize("scale", [1e9, 1e-20])
def test_shares_at_extreme_scales(F, scale):
    """A share in which some rows of a wave see no key and others do, at scales that take the initial
    maximum (-1e30) past the range of fp32, and close to zero.  Scores have a spread of about 3 either way."""
    B, H, Sq, Skv, dh = 1, 4, 300, 1300, 64
    std = math.sqrt(3.0 / (scale * math.sqrt(dh)))
    q = I.normal(74, 0, "q", (B, H, Sq, dh), std, bf16=True)
    k = I.normal(74, 0, "k", (B, H, Skv, dh), std, bf16=True)
    v = I.normal(74, 0, "v", (B, H, Skv, dh), 1.0, bf16=True)
    need = F.forge_attn_fused_workspace_bytes(B, H, H, Sq, Skv, dh, torch.bfloat16)
    assert need > 0
    for ws in (F.workspace(need), None):
        out = torch.empty(B, Sq, H * dh, dtype=torch.bfloat16, device="cuda")
        F.forge_attn_fused(dev(q, True), dev(k, True), dev(v, True), out, scale=scale, causal=True, workspace=ws)
        torch.cuda.synchronize()
        check(out, O.attention(q, k, v, scale, True), True, "scale %g, shares %s" % (scale, ws is not None))
