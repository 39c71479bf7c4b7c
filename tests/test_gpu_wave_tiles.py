"""bf16 linears on shared slabs with tiles of 48 rows or columns: edges of the tiles, one, two, three and more slabs per wave, all
epilogues, padded and odd row strides, the head split of a short prompt."""
import math

import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act,use_b,use_r", [("none", True, True), ("gelu_tanh", True, False), ("swiglu", True, True), ("silu", False, True)])
@pytest.mark.parametrize("tile,M,N,K,ld", [
    ("2,3", 128, 3072, 768, 0), ("2,3", 97, 3000, 512, 0), ("2,3", 127, 2875, 576, 2880),          # 32 x 48
    ("3,2", 128, 2304, 768, 0), ("3,2", 143, 2272, 1088, 0), ("3,2", 97, 2299, 1472, 2304),        # 48 x 32
    ("3,3", 186, 3072, 768, 0), ("3,3", 145, 3017, 1088, 3024), ("3,3", 190, 2976, 448, 0),        # 48 x 48
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
