"""Scratch of single-query attention: the reported size serves shorter caches and smaller batches, of the operator and of whole
models, and no call is refused for bytes that its launch does not write."""
import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import binding as F
from paper_2604_16498_amd import inputs as I
from test_plan_host import fake_model
from util import check, dev, dev_dict

HEADS = [(12, 12, 64), (16, 16, 128), (32, 8, 128), (32, 32, 128), (32, 2, 128), (25, 25, 64), (300, 300, 64)]


def size(B, hq, hkv, kv, dh):
    return F.forge_attn_fused_workspace_bytes(B, hq, hkv, 1, kv, dh, torch.bfloat16)


@pytest.mark.parametrize("hq,hkv,dh", HEADS)
@pytest.mark.parametrize("kv", [1, 300, 511, 512, 1500, 8192])
def test_a_size_serves_smaller_batches(hq, hkv, dh, kv):
    sizes = [size(B, hq, hkv, kv, dh) for B in range(1, 70)]
    assert sizes == sorted(sizes)
    assert kv >= 512 or max(sizes) == 0                 # never cut


@pytest.mark.parametrize("shape", [I.GPT2_SMALL, I.OPT_1P3B, I.LLAMA_8B], ids=["768", "2048", "4096"])
def test_a_model_sized_for_one_sequence_more(shape):
    m = fake_model(shape, 2, False, F.FORGE_BF16)
    for cap in (256, 400, 1500, 8192):
        sizes = [F.forge_model_workspace_bytes(m, B, 1, cap) for B in range(1, 18)]
        assert sizes == sorted(sizes), cap              # (past 16 rows the projections have fewer planes)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,dh,kv,given", [
    (8, 12, 12, 64, 300, "none"), (2, 16, 4, 128, 511, "none"),     # shorter than any range is cut
    (16, 8, 8, 128, 1500, "for 24 sequences"),
    (1, 32, 8, 128, 700, "for 5 sequences"),
    (2, 64, 1, 128, 8192, "the library's"),                        # a group of the vector-ALU kernel, which writes no partials
])
def test_calls_that_need_no_more(B, Hq, Hkv, dh, kv, given):
    q = I.normal(91, 0, "q", (B, Hq, 1, dh), 1.0, bf16=True)
    k, v = (I.normal(91, 0, n, (B, Hkv, kv, dh), 1.0, bf16=True) for n in ("k_cache", "v_cache"))
    ref = O.attention(q, k, v, dh ** -0.5, True)
    pos = torch.full((B,), kv - 1, dtype=torch.int32, device="cuda")
    tq, tk, tv = dev(q, True), dev(k, True), dev(v, True)
    ws = F.workspace(size(int(given.split()[1]), Hq, Hkv, kv, dh)) if given.startswith("for") else None
    calls = [lambda out: F.forge_attn_fused(tq, tk, tv, out, kv, causal=True, workspace=ws),
             lambda out: F.forge_attn_decode_varlen(tq, tk, tv, out, pos, kv - 1, workspace=ws)]
    if given == "the library's":
        calls = [lambda out: F.forge_attn_decode_static(tq, tk, tv, out, kv)]
    for call in calls:
        out = torch.full((B, 1, Hq * dh), 7.0, dtype=torch.bfloat16, device="cuda")
        call(out)
        torch.cuda.synchronize()
        check(out, ref, True, "B=%d heads %d/%d kv %d, workspace: %s" % (B, Hq, Hkv, kv, given))


@pytest.mark.gpu
def test_layer_of_a_batch_that_is_never_cut():
    """48 sequences of 12 heads fill the chip with one block each: a layer over 600 rows runs in the workspace of one over 500."""
    sh, B, cap = I.GPT2_SMALL, 48, 600
    desc = F.make_block_desc(sh, dev_dict(I.block_weights(sh, 92, 0, bf16=True, weight_std=0.05), True))
    pos = torch.arange(cap - B, cap, dtype=torch.int32, device="cuda")
    x = dev(I.normal(92, 0, "x", (B, 1, sh.d_model), 1.0, bf16=True), True)
    outs = []
    for rows in (cap, 500):
        kv = [dev(I.normal(92, 0, n, (B, sh.kv_heads, cap, sh.head_dim), 1.0, bf16=True), True) for n in ("k_cache", "v_cache")]
        outs.append(torch.empty_like(x))
        ws = F.workspace(F.forge_decoder_block_workspace_bytes(desc, B, 1, rows))
        F.forge_decoder_block_decode(desc, x, outs[-1], *kv, pos, cap - 1, ws)
    torch.cuda.synchronize()
    assert torch.equal(*outs)
