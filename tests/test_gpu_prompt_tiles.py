"""Tiles of the persistent kernel by the length of a prompt: the 192 x 256 tile at the edges of its rows and columns, with every
epilogue, and with the head split and rotation of a layer's QKV projection; 128-tiles over whole reductions."""
import math

import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,ld,act,use_b,use_r,tile", [
    (1345, 5896, 2048, 0, "none", True, True, "192,256,2,4"),           # one row in the last tile, 8 columns in the last
    (1344, 6140, 1600, 6144, "gelu_tanh", True, False, "192,256,2,4"),  # whole row tiles, ragged columns of padded rows
    (1343, 6144, 1600, 0, "none", False, True, "192,256,2,4"),          # one row short
    (346, 11080, 2048, 0, "swiglu", True, True, "192,256,2,4"),         # gated: 128 output columns a tile, 72 in the last
    (1195, 2056, 2048, 0, "none", True, True, "128,128,2,4"),           # not cut along K
])
def test_linear_tiles(M, N, K, ld, act, use_b, use_r, tile):
    from paper_2604_16498_amd import binding as F
    wn = 2 * N if act == "swiglu" else N
    ldy = ld or N
    assert F.forge_gemm_variant(M, N, K, act, torch.bfloat16, ldy=ldy) == "gemm_bf16_pers<%s>" % tile
    x = I.normal(65, 0, "x", (M, K), 1.0, bf16=True)
    w = I.normal(65, 0, "w_up", (wn, K), 1.0 / math.sqrt(K), bf16=True)
    b = I.normal(65, 0, "b_up", (wn,), 0.5, bf16=True) if use_b else None
    r = I.normal(65, 0, "residual", (M, ldy), 1.0, bf16=True) if use_r else None
    ref = O.gemm_bias_act(x, w, b, None if r is None else r[:, :N], act)
    ty = torch.full((M, ldy), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = F.workspace(F.forge_gemm_workspace_bytes(M, N, K, act, torch.bfloat16))
    F.forge_gemm_bias_gelu(dev(x, True), dev(w, True), dev(b, True), dev(r, True), ty, act, ws, n=N)
    torch.cuda.synchronize()
    check(ty[:, :N], ref, True, "%dx%dx%d %s" % (M, N, K, act))
    assert torch.all(ty[:, N:] == 7.0)


@pytest.mark.parametrize("batch,seq,q_heads,dh", [
    (1, 1300, 32, 128),        # 192 x 256 tiles, a head half a tile
    (2, 647, 64, 64),          # 192 x 256 tiles over two sequences, one ending inside a tile
    (1, 777, 16, 128),         # 128 x 128 tiles
])
def test_rotated_heads(batch, seq, q_heads, dh):
    """The K and V rows that a layer writes to its cache against the oracle's norm, projection and rotation."""
    from paper_2604_16498_amd import binding as F
    d, kv = 2048, q_heads // 4
    sh = I.BlockShape(d, q_heads, kv, dh, 704, norm="rmsnorm", mlp_act="swiglu", use_rope=True, rope_base=10000.0,
                      has_bias=False)
    w = I.block_weights(sh, 66, 0, bf16=True, random_affine=True)
    x = I.normal(66, 0, "x", (batch, seq, d), 1.0, bf16=True)
    cap = (seq + 63) // 64 * 64
    tw = {k: dev(v, True) for k, v in w.items()}
    desc = F.make_block_desc(sh, tw)
    tk, tv = (torch.full((batch, kv, cap, dh), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    tx = dev(x, True)
    ws = F.workspace(F.forge_decoder_block_workspace_bytes(desc, batch, seq, cap))
    F.forge_decoder_block(desc, tx, torch.empty_like(tx), tk, tv, 0, ws)
    y = torch.empty_like(tx)
    F.forge_residual_norm(tx, None, tw["norm1_g"], None, None, y, sh.eps, sh.norm)
    torch.cuda.synchronize()
    R = sorted({0, 1, 127, 128, 191, 192, 255, 383, 384, 575, 576, seq - 1} & set(range(seq)))
    for b in range(batch):
        rows = O.linear(host(y[b, R]), w["w_qkv"], None).reshape(len(R), -1, dh).transpose(1, 0, 2)
        k, v = rows[q_heads:q_heads + kv], rows[q_heads + kv:]
        check(tk[b][:, R], O.rope(k, np.asarray(R), sh.rope_base), True, "k rows")
        check(tv[b][:, R], v, True, "v rows")
    assert torch.all(tk[:, :, seq:] == 7.0) and torch.all(tv[:, :, seq:] == 7.0)
