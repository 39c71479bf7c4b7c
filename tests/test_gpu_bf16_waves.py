"""bf16 linears whose k slabs are shared by the waves of a block: edges of the tiles (16, 32 and 64 rows of x and of the
weight), one slab, a slab for each of the 8 waves and one more, all epilogues, padded and odd row strides."""
import math

import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act,use_b,use_r", [("none", True, True), ("gelu_tanh", True, False), ("swiglu", True, True),
                                             ("silu", False, True)])
@pytest.mark.parametrize("M,N,K,ld", [
    (1, 8, 64, 0), (15, 40, 64, 0), (17, 1001, 512, 1008), (33, 515, 576, 0),            # decode-sized, odd widths
    (64, 4096, 1088, 0), (63, 2056, 2048, 0), (40, 8192, 128, 0),
    (65, 24, 64, 0), (66, 776, 576, 0), (127, 2304, 768, 0), (129, 768, 3072, 0),        # prompts against few weight rows
    (257, 515, 128, 520), (300, 1001, 1152, 1008), (255, 2048, 2048, 0), (385, 2312, 640, 0),
    (513, 1536, 4096, 0),
])
def test_linear_shared_slabs(M, N, K, ld, act, use_b, use_r):
    from paper_2604_16498_amd import binding as F
    wn = 2 * N if act == "swiglu" else N
    ldy = ld or N
    x = I.normal(64, 0, "x", (M, K), 1.0, bf16=True)
    w = I.normal(64, 0, "w_up", (wn, K), 1.0 / math.sqrt(K), bf16=True)
    b = I.normal(64, 0, "b_up", (wn,), 0.5, bf16=True) if use_b else None
    r = I.normal(64, 0, "residual", (M, ldy), 1.0, bf16=True) if use_r else None
    ref = O.gemm_bias_act(x, w, b, None if r is None else r[:, :N], act)
    ty = torch.full((M, ldy), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = F.workspace(F.forge_gemm_workspace_bytes(M, N, K, act, torch.bfloat16))
    F.forge_gemm_bias_gelu(dev(x, True), dev(w, True), dev(b, True), dev(r, True), ty, act, ws, n=N)
    torch.cuda.synchronize()
    check(ty[:, :N], ref, True, "%dx%dx%d %s" % (M, N, K, act))
    assert torch.all(ty[:, N:] == 7.0)
