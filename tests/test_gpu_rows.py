"""GPU parity of the linear that keeps the rows of x in registers (decode steps, some prompts), at the sizes where its
tiles (16 weight rows, 8 waves that share K, groups of 16 rows of x, up to 8 collected tiles) have
remainders, against the fp64 oracle.  Prompts: its two chunks of 64 rows, what takes the others, and the bf16 copy of an int8 weight."""
import math

import numpy as np
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev, dev_dict

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2604_16498_amd import binding
    binding.lib()
    return binding


CASES = [  # M, N, K, act, residual, padded row stride
    (1, 8, 64, "none", True, 0),               # half a tile, two steps for eight waves
    (16, 40, 192, "gelu_erf", False, 0),       # six steps, a ragged second tile
    (17, 1003, 832, "relu", True, 1008),       # one row past a group, odd columns in a padded stride
    (32, 24, 1088, "swiglu", False, 0),        # 34 steps: the last waves have fewer
    (33, 8200, 2048, "silu", True, 0),         # past two groups
    (64, 776, 1920, "swiglu", False, 0),
    (5, 8200, 4096, "none", False, 0),         # the longest single range; more tiles than blocks
    (16, 33000, 256, "gelu_tanh", False, 0),   # more than 8 tiles per block: the sums are collected twice
    (24, 33000, 2048, "gelu_tanh", False, 0),  # ... with two groups of x rows
    (17, 1003, 1280, "swiglu", True, 1008),    # 5, 9 and 10 steps per wave (int8: 3, 5 and 5)
    (40, 776, 1280, "swiglu", False, 0),
    (20, 1003, 2304, "swiglu", True, 1008),
    (30, 776, 2560, "swiglu", False, 0),
    (7, 2048, 8192, "gelu_tanh", True, 0),     # several k ranges and the reduce launch
    (40, 768, 3072, "swiglu", True, 0),
    (9, 520, 4160, "swiglu", False, 0),        # one step past a single range
    # prompts in two chunks of 64 rows: ragged second chunks, odd columns in a padded stride, a ragged last tile, gated
    (105, 8203, 2048, "silu", True, 8208),
    (99, 10248, 1280, "relu", False, 0),
    (114, 6144, 1280, "swiglu", True, 0),
    (127, 10248, 1024, "none", True, 0),
    # other prompts (int8: the bf16 copy on the tile kernels)
    (65, 2304, 768, "none", False, 0),
    (129, 1003, 704, "gelu_tanh", True, 1008),
    (300, 768, 768, "swiglu", False, 0),
    (130, 2056, 2048, "relu", True, 0),
    (200, 768, 3072, "none", True, 0),
]
OTHERS = [c[:3] for c in CASES[-5:]]


@pytest.mark.parametrize("w8", [False, True], ids=["bf16", "int8"])
@pytest.mark.parametrize("M,N,K,act,use_r,ld", CASES)
def test_rows_linear(F, M, N, K, act, use_r, ld, w8):
    if w8 and K % 128 != 0:
        K += 64
    wn = 2 * N if act == "swiglu" else N
    ldy = ld or N
    x = I.normal(71, 0, "x", (M, K), 1.0, bf16=True)
    w = I.normal(71, 0, "w_up", (wn, K), 1.0 / math.sqrt(K), bf16=True)
    b = I.normal(71, 0, "b_up", (wn,), 0.5, bf16=True)
    r = I.normal(71, 0, "residual", (M, ldy), 1.0, bf16=True) if use_r else None
    q, s = O.quantize_int8(w) if w8 else (None, None)
    ref = O.gemm_bias_act(x, O.dequantize_int8(q, s) if w8 else w, b, None if r is None else r[:, :N], act)
    tx, tb, tr = dev(x, True), dev(b, True), None if r is None else dev(r, True)
    tw = torch.from_numpy(q).cuda() if w8 else dev(w, True)
    ts = torch.from_numpy(s).cuda() if w8 else None
    if not w8:
        kernel = "gemm_bf16_waves" if (M, N, K) in OTHERS else "gemm_bf16_rows"
        assert kernel in F.forge_gemm_variant(M, N, K, act, torch.bfloat16, ldy=ldy)
    need = F.forge_gemm_w8_workspace_bytes(M, N, K, act) if w8 else F.forge_gemm_workspace_bytes(M, N, K, act, torch.bfloat16)
    outs = []
    for _ in range(2):
        ty = torch.full((M, ldy), 7.0, dtype=torch.bfloat16, device="cuda")
        if w8:
            F.forge_gemm_w8(tx, tw, ts, tb, tr, ty, act, F.workspace(max(need, 256)), n=N)
        else:
            F.forge_gemm_bias_gelu(tx, tw, tb, tr, ty, act, F.workspace(need), n=N)
        outs.append(ty)
    torch.cuda.synchronize()
    check(outs[0][:, :N], ref, True, "rows linear %s %dx%dx%d" % (act, M, N, K))
    assert torch.all(outs[0][:, N:] == 7.0)
    assert torch.equal(outs[0], outs[1])


def test_positions_rotate_like_fp64(F):
    """The rotated head split at positions up to 60000 against the fp64 definition: every new row of the
    k cache, one linear and one rotation away from x (bf16 rounding of the output is all that is left)."""
    sh = I.BlockShape(d_model=256, q_heads=4, kv_heads=2, head_dim=128, d_ff=256, norm="rmsnorm", mlp_act="swiglu",
                      use_rope=True, rope_base=500000.0, has_bias=False)
    B, cap = 20, 60001
    pos = [int(60000 * (i / (B - 1)) ** 2) for i in range(B)]
    w = I.block_weights(sh, 72, 0, bf16=True)
    x = I.normal(72, 0, "x", (B, 1, sh.d_model), 1.0, bf16=True)
    tw = dev_dict(w, True)
    desc = F.make_block_desc(sh, tw)
    tx = dev(x, True)
    tk, tv = (torch.zeros(B, sh.kv_heads, cap, sh.head_dim, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    out = torch.empty_like(tx)
    tpos = torch.tensor(pos, dtype=torch.int32, device="cuda")
    F.forge_decoder_block_decode(desc, tx, out, tk, tv, tpos, max(pos), F.workspace(F.forge_decoder_block_workspace_bytes(desc, B, 1, cap)))
    got = torch.stack([tk[b, :, p] for b, p in enumerate(pos)])
    want = []
    nq, nk = sh.q_heads * sh.head_dim, sh.kv_heads * sh.head_dim
    for b, p in enumerate(pos):
        y = O.rms_norm(x[b], w["norm1_g"], sh.eps)
        k = O.linear(y, w["w_qkv"][nq:nq + nk]).reshape(1, sh.kv_heads, 1, sh.head_dim)
        want.append(O.rope(k, np.array([p]), sh.rope_base)[0, :, 0])
    check(got, np.stack(want), True, "rotated k rows", chain=True)

