"""fp32 linears whose k slabs are shared by the waves of a block: edges of the tiles (32 rows, 16 or 32 weight
rows, 32-element slabs dealt to 8 waves), few and many tiles, the gated form."""
import math

import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act,use_b,use_r", [("none", True, True), ("gelu_tanh", True, False), ("swiglu", True, True),
                                             ("silu", False, True)])
@pytest.mark.parametrize("M,N,K", [
    (1, 1, 4), (31, 15, 28), (32, 16, 32), (33, 17, 36), (65, 33, 252), (64, 31, 260),   # tile and slab edges
    (40, 770, 768), (128, 2304, 768), (250, 1530, 772),                                  # one round of tiles, several
    (17, 768, 3072), (200, 770, 3076), (33, 1100, 4100),                                 # slabs past what a wave holds in flight
])
def test_f32_linear_shared_slabs(M, N, K, act, use_b, use_r):
    from paper_2604_16498_amd import binding as F
    assert "waves" in F.forge_gemm_variant(M, N, K, act, torch.float32)
    wn = 2 * N if act == "swiglu" else N
    x = I.normal(63, 0, "x", (M, K), 1.0, bf16=False)
    w = I.normal(63, 0, "w_up", (wn, K), 1.0 / math.sqrt(K), bf16=False)
    b = I.normal(63, 0, "b_up", (wn,), 0.5, bf16=False) if use_b else None
    r = I.normal(63, 0, "residual", (M, N), 1.0, bf16=False) if use_r else None
    ref = O.gemm_bias_act(x, w, b, r, act)
    tx, tw, tb, tr = (dev(a, False) for a in (x, w, b, r))
    ty = torch.full((M, N), 7.0, device="cuda")
    ws = F.workspace(F.forge_gemm_workspace_bytes(M, N, K, act, torch.float32))
    F.forge_gemm_bias_gelu(tx, tw, tb, tr, ty, act, ws)
    torch.cuda.synchronize()
    err = abs(host(ty) - ref)
    # a sum of K products carries at most ~K/16 roundings one after the other (16 partial sums or more) of a
    # partial sum of order 1: 2^-24 (K/16 + 30) with the epilogue's, twice that for a gated product
    bound = 2.0 ** -24 * (K / 16 + 30) * (1.0 + abs(ref).max()) * (2.0 if act == "swiglu" else 1.0)
    assert err.max() <= bound, (err.max(), bound)
