"""fp32 linears on shared slabs with tiles of 32 x 48: edges of the tile, slabs in flight and past them, every epilogue that takes it."""
import math

import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act,use_b,use_r", [("none", True, True), ("gelu_tanh", True, False), ("silu", False, True)])
@pytest.mark.parametrize("M,N,K", [(128, 2304, 768), (127, 3070, 772), (97, 3025, 500), (512, 767, 1028)])
def test_f32_tiles_of_48(M, N, K, act, use_b, use_r):
    from paper_2604_16498_amd import binding as F
    assert F.forge_gemm_variant(M, N, K, act, torch.float32) == "gemm_f32_waves<3>"
    x = I.normal(66, 0, "x", (M, K), 1.0, bf16=False)
    w = I.normal(66, 0, "w_up", (N, K), 1.0 / math.sqrt(K), bf16=False)
    b = I.normal(66, 0, "b_up", (N,), 0.5, bf16=False) if use_b else None
    r = I.normal(66, 0, "residual", (M, N), 1.0, bf16=False) if use_r else None
    ref = O.gemm_bias_act(x, w, b, r, act)
    ty = torch.full((M, N), 7.0, device="cuda")
    ws = F.workspace(max(16, F.forge_gemm_workspace_bytes(M, N, K, act, torch.float32)))
    F.forge_gemm_bias_gelu(*(dev(a, False) for a in (x, w, b, r)), ty, act, ws)
    torch.cuda.synchronize()
    err = abs(host(ty) - ref)
    # at most K / 16 roundings one after the other (16 partial sums or more) of a partial sum of order 1, and the epilogue's
    bound = 2.0 ** -24 * (K / 16 + 30) * (1.0 + abs(ref).max())
    assert err.max() <= bound, (err.max(), bound)


@pytest.mark.parametrize("M,N,K,n", [(128, 2304, 768, 768), (97, 3025, 500, 70), (512, 767, 1028, 48), (512, 768, 3072, 48)])
def test_sums_as_on_the_narrow_tiles(M, N, K, n):
    """The same partial sums in the same order as tiles of 32 x 16: equal bit for bit, so no larger an error."""
    from paper_2604_16498_amd import binding as F
    assert F.forge_gemm_variant(M, N, K, "none", torch.float32) == "gemm_f32_waves<3>"
    assert F.forge_gemm_variant(M, n, K, "none", torch.float32) == "gemm_f32_waves<1>"
    x = dev(I.normal(67, 0, "x", (M, K), 1.0, bf16=False), False)
    w = dev(I.normal(67, 0, "w_up", (N, K), 1.0 / math.sqrt(K), bf16=False), False)
    wide, narrow = (torch.full((M, c), 7.0, device="cuda") for c in (N, n))
    for y in (wide, narrow):
        F.forge_gemm_bias_gelu(x, w[:y.shape[1]].contiguous(), None, None, y, "none", F.workspace(16))
    torch.cuda.synchronize()
    assert torch.equal(wide[:, :n], narrow)
