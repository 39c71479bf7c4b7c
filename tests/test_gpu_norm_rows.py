"""Residual + norm with a whole row's loads in flight: rows past the last wave of a block, widths that leave lanes and chunks
without elements, every combination of delta, shift and stored sum, and the sum stored over the rows that it is of."""
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import inputs as I
from util import check, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("kind,use_delta,use_beta,use_h", [("layernorm", False, True, False), ("layernorm", True, False, True),
                                                           ("rmsnorm", True, False, True), ("rmsnorm", False, False, False)])
@pytest.mark.parametrize("rows,d", [(1, 8), (3, 512), (5, 520), (129, 1016), (1025, 2040), (2, 1032), (7, 4088), (3, 8184), (2, 16376)])
def test_norm_rows(rows, d, kind, use_delta, use_beta, use_h, bf16):
    from paper_2604_16498_amd import binding as F
    x = I.normal(67, 0, "x", (rows, d), 1.0, bf16=bf16)
    delta = I.normal(67, 0, "residual", (rows, d), 1.0, bf16=bf16) if use_delta else None
    g = I.normal(67, 0, "norm1_g", (d,), 1.0, bf16=bf16)
    b = I.normal(67, 0, "norm1_b", (d,), 1.0, bf16=bf16) if use_beta else None
    h_ref, y_ref = O.residual_norm(x, delta, g, b, 1e-5, kind)
    dt = torch.bfloat16 if bf16 else torch.float32
    whole_y, whole_h = (torch.full((rows + 1, d), 7.0, dtype=dt, device="cuda") for _ in range(2))
    F.forge_residual_norm(dev(x, bf16), dev(delta, bf16), dev(g, bf16), dev(b, bf16), whole_h[:rows] if use_h else None,
                          whole_y[:rows], 1e-5, kind)
    torch.cuda.synchronize()
    check(whole_y[:rows], y_ref, bf16, "%d x %d %s" % (rows, d, kind))
    if use_h:
        check(whole_h[:rows], h_ref, bf16, "stored sum")
    assert torch.all(whole_y[rows:] == 7.0) and torch.all(whole_h[rows:] == 7.0)


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("rows,d", [(3, 512), (129, 1016), (1025, 2040), (7, 4088), (2, 16376)])    # one wave per row, one block per row
def test_sum_over_its_own_rows(rows, d, bf16):
    from paper_2604_16498_amd import binding as F
    x = I.normal(67, 0, "x", (rows, d), 1.0, bf16=bf16)
    delta = I.normal(67, 0, "residual", (rows, d), 1.0, bf16=bf16)
    g = I.normal(67, 0, "norm1_g", (d,), 1.0, bf16=bf16)
    h_ref, y_ref = O.residual_norm(x, delta, g, None, 1e-5, "rmsnorm")
    tx, ty = dev(x, bf16), torch.empty(rows, d, dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
    F.forge_residual_norm(tx, dev(delta, bf16), dev(g, bf16), None, tx, ty, 1e-5, "rmsnorm")
    torch.cuda.synchronize()
    check(ty, y_ref, bf16, "%d x %d" % (rows, d))
    check(tx, h_ref, bf16, "stored sum")
