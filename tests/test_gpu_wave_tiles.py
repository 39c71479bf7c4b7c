"""bf16 linears on shared slabs with tiles of 48 rows or columns: edges of the tiles, one to five slabs per wave,
all epilogues, padded and odd row strides, the head split of a short prompt."""
import math

import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev, dev_dict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act,use_b,use_r", [("none", True, True), ("gelu_tanh", True, False), ("swiglu", True, True), ("silu", False, True)])
@pytest.mark.parametrize("tile,M,N,K,ld", [
    ("2,3", 128, 3072, 768, 0), ("2,3", 97, 3000, 512, 0), ("2,3", 127, 2875, 576, 2880),          # 32 x 48
    ("3,2", 128, 2304, 768, 0), ("3,2", 143, 2272, 1088, 0), ("3,2", 97, 2299, 1472, 2304),        # 48 x 32
    ("3,3", 186, 3072, 768, 0), ("3,3", 145, 3017, 1088, 3024), ("3,3", 190, 2976, 448, 0),        # 48 x 48
    # the back edge of the slab loop: four slabs per wave, four and five
    ("2,3", 97, 3000, 2048, 0), ("2,3", 128, 3056, 2304, 0), ("3,2", 143, 2272, 2048, 0), ("3,2", 128, 2304, 2304, 2312),
    ("3,3", 68, 6144, 2048, 0), ("3,3", 145, 3024, 2304, 3032),
])
def test_tiles_of_48(tile, M, N, K, ld, act, use_b, use_r):
    from paper_2604_16498_amd import binding as F
    wn = N // 16 * 16 if act == "swiglu" else N                  # weight rows: the plan counts these
    N, ldy = (wn // 2, wn // 2) if act == "swiglu" else (N, ld or N)
    assert F.forge_gemm_variant(M, N, K, act, torch.bfloat16, ldy=ldy) == "gemm_bf16_waves<%s>" % tile
    x = I.normal(65, 0, "x", (M, K), 1.0, bf16=True)
    w = I.normal(65, 0, "w_up", (wn, K), 1.0 / math.sqrt(K), bf16=True)
    b = I.normal(65, 0, "b_up", (wn,), 0.5, bf16=True) if use_b else None
    r = I.normal(65, 0, "residual", (M, ldy), 1.0, bf16=True) if use_r else None
    ref = O.gemm_bias_act(x, w, b, None if r is None else r[:, :N], act)
    ty = torch.full((M, ldy), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = F.workspace(max(16, F.forge_gemm_workspace_bytes(M, N, K, act, torch.bfloat16)))
    F.forge_gemm_bias_gelu(dev(x, True), dev(w, True), dev(b, True), dev(r, True), ty, act, ws, n=N)
    torch.cuda.synchronize()
    check(ty[:, :N], ref, True, "%dx%dx%d %s" % (M, N, K, act))
    assert torch.all(ty[:, N:] == 7.0)


@pytest.mark.parametrize("act,use_b,use_r", [("none", True, True), ("gelu_tanh", True, False), ("silu", False, True)])
@pytest.mark.parametrize("tile,M,N,K,ld", [
    ("2,3", 64, 6144, 1024, 0), ("2,3", 57, 4493, 2304, 4497), ("2,3", 50, 4301, 3072, 4301),
    ("3,2", 33, 7079, 1088, 7081), ("3,2", 48, 8192, 2048, 0), ("3,2", 47, 5075, 1024, 5076),
])
def test_tiles_of_48_few_rows(tile, M, N, K, ld, act, use_b, use_r):
    """At most 64 rows, where x in registers is the alternative: outputs element by element where the stride is odd."""
    test_tiles_of_48(tile, M, N, K, ld, act, use_b, use_r)


@pytest.mark.parametrize("tile,B,S,pos0,heads", [("3,2", 1, 128, 0, 12), ("2,3", 2, 64, 37, 16), ("3,3", 2, 93, 5, 16)])
def test_head_split_on_tiles_of_48(tile, B, S, pos0, heads):
    from paper_2604_16498_amd import binding as F
    sh = I.BlockShape(768, heads, heads, 64, 256)
    assert F.forge_gemm_variant(B * S, sh.qkv_out, 768, "none", torch.bfloat16) == "gemm_bf16_waves<%s>" % tile
    cap = pos0 + S + 3
    w = I.block_weights(sh, 68, 0, bf16=True, bias_std=0.05, random_affine=True, weight_std=0.04)
    x = I.normal(68, 0, "x", (B, S, 768), 1.0, bf16=True)
    kc, vc = (np.zeros((B, heads, cap, 64), np.float32) for _ in range(2))
    for c, name in ((kc, "k_cache"), (vc, "v_cache")):
        c[:, :, :pos0] = I.normal(68, 0, name, (B, heads, pos0, 64), 1.0, bf16=True)
    tk, tv = dev(kc, True), dev(vc, True)
    kc, vc = kc.astype(np.float64), vc.astype(np.float64)
    ref = O.decoder_block(sh, w, x, kc, vc, pos0=pos0)
    tw = dev_dict(w, True)                     # (the descriptor holds raw pointers)
    desc = F.make_block_desc(sh, tw)
    out = torch.empty(B, S, 768, dtype=torch.bfloat16, device="cuda")
    F.forge_decoder_block(desc, dev(x, True), out, tk, tv, pos0, F.workspace(F.forge_decoder_block_workspace_bytes(desc, B, S, cap)))
    torch.cuda.synchronize()
    check(tk, kc, True, "k cache")
    check(tv, vc, True, "v cache")
    check(out, ref, True, "layer", chain=True)
