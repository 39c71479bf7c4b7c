"""bf16 linears whose k slabs are shared by the waves of a block: edges of the tiles (16, 32 and 64 rows of x and of the
weight), one slab, a slab for each of the 8 waves and one more, all epilogues, padded and odd row strides.  Every case
names the kernel that takes it, so that a rule which sends it elsewhere is seen."""
import math

import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev

pytestmark = pytest.mark.gpu


def _epilogues(gated):
    return [("none", True, True), ("gelu_tanh", True, False), ("silu", False, True)] + ([("swiglu", True, True)] if gated else [])


@pytest.mark.parametrize("M,N,K,ld,act,use_b,use_r", [(*c, *e) for c, gated in [
    # decode-sized: one row, odd widths and strides (element-wise outputs), two row blocks
    ((1, 40, 1024, 0), False), ((15, 1001, 1088, 1003), False), ((33, 515, 2048, 0), False), ((64, 1544, 1088, 0), False),
    ((63, 1030, 4096, 1036), False), ((17, 1602, 1152, 0), False),
    # prompts against few weight rows, tiles of 16 x 16 to 64 x 64
    ((65, 24, 64, 0), True), ((66, 776, 576, 0), True), ((127, 2304, 768, 0), True), ((129, 768, 3072, 0), True),
    ((257, 515, 128, 520), False), ((300, 1001, 1152, 1008), False), ((255, 2048, 2048, 0), True), ((383, 2312, 640, 0), False),
    ((513, 1536, 4096, 0), False),
] for e in _epilogues(gated)])
def test_linear_shared_slabs(M, N, K, ld, act, use_b, use_r):
    from paper_2604_16498_amd import binding as F
    assert F.forge_gemm_variant(M, N, K, act, torch.bfloat16, ldy=ld or N).startswith("gemm_bf16_waves<")
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
