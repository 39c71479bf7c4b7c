"""The reduce launch of linears cut along K: whole rows in groups of 4 columns, and rows that are not (odd widths, odd row
strides), in prompts and decode-sized problems, with every epilogue."""
import math

import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_b,use_r", [(True, True), (False, False)])
@pytest.mark.parametrize("M,N,K,ld,act", [
    (100, 4104, 4096, 0, "none"), (200, 4104, 4096, 4112, "gelu_tanh"), (130, 2056, 8192, 0, "swiglu"),
    (17, 4100, 8192, 0, "none"), (17, 4100, 8192, 4102, "none"), (33, 4098, 8192, 4104, "gelu_tanh"), (8, 2052, 8192, 0, "swiglu"),
])
def test_split_reduce(M, N, K, ld, act, use_b, use_r):
    from paper_2604_16498_amd import binding as F
    wn = 2 * N if act == "swiglu" else N
    ldy = ld or N
    assert F.forge_gemm_variant(M, N, K, act, torch.bfloat16, ldy=ldy).endswith("+splitk")
    x = I.normal(68, 0, "x", (M, K), 1.0, bf16=True)
    w = I.normal(68, 0, "w_up", (wn, K), 1.0 / math.sqrt(K), bf16=True)
    b = I.normal(68, 0, "b_up", (wn,), 0.5, bf16=True) if use_b else None
    r = I.normal(68, 0, "residual", (M, ldy), 1.0, bf16=True) if use_r else None
    ref = O.gemm_bias_act(x, w, b, None if r is None else r[:, :N], act)
    ty = torch.full((M, ldy), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = F.workspace(F.forge_gemm_workspace_bytes(M, N, K, act, torch.bfloat16))
    F.forge_gemm_bias_gelu(dev(x, True), dev(w, True), dev(b, True), dev(r, True), ty, act, ws, n=N)
    torch.cuda.synchronize()
    check(ty[:, :N], ref, True, "%dx%dx%d %s" % (M, N, K, act))
    assert torch.all(ty[:, N:] == 7.0)
