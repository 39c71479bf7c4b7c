"""Workspace of layers, models and compiled models for prompts: the attention's key shares get no bytes of their own,
so a size does not grow with the cache, and a buffer for a longer prompt serves a shorter one; and with a
buffer of exactly the reported size the shares are cut (plain and compiled alike) without a byte written outside."""
import pytest
import torch

from oracle import forge_oracle as O
from paper_2604_16498_amd import binding as B
from paper_2604_16498_amd import inputs as I
from test_plan_host import fake_model
from util import check, dev, dev_dict

SHAPES = {"768": I.GPT2_SMALL, "2048": I.OPT_1P3B, "4096": I.LLAMA_8B}


@pytest.mark.parametrize("shape,shorter,longer", [
    ("2048", 2048, 4096), ("4096", 1024, 2048), ("4096", 300, 500), ("768", 777, 1024), ("4096", 80, 777),
])
@pytest.mark.parametrize("w8", [False, True], ids=["bf16", "int8"])
def test_a_buffer_for_the_longer_prompt_serves_the_shorter(shape, shorter, longer, w8):
    m = fake_model(SHAPES[shape], 2, False, B.FORGE_BF16, w8=w8)
    block = lambda S, cap: B.forge_decoder_block_workspace_bytes(m.layers[0], 1, S, cap)
    model = lambda S, cap: B.forge_model_workspace_bytes(m, 1, S, cap)
    compiled = lambda S, pos: B.CompiledModel(m, 1, S, pos, S + pos).workspace_bytes()
    for size in (block, model):
        assert 0 < size(shorter, 8192) <= size(longer, 8192)
        assert size(shorter, shorter) == size(shorter, 8192) and size(longer, longer) == size(longer, 8192)
    assert compiled(shorter, 0) == compiled(shorter, 4000) <= compiled(longer, 4000)


@pytest.mark.parametrize("N,K,act", [(768, 4100, "none"), (320, 8192, "swiglu"), (64, 16384, "none")])
def test_an_fp32_size_serves_the_cut_reductions_of_fewer_rows(N, K, act):
    size = lambda M: B.forge_gemm_workspace_bytes(M, N, K, act, torch.float32)
    cut = 16 // -(-N // 64) * 64                  # up to here a reduction of more than 3072 is cut
    assert 0 < size(cut)
    assert all(size(M) >= size(cut) for M in range(cut + 1, 4 * cut, 37))


@pytest.mark.gpu
@pytest.mark.parametrize("d,hq,hkv,dh,ff,llama,S,pos", [
    (512, 4, 2, 128, 1408, True, 80, 1500),      # shares in the MLP rows and the GEMM planes
    (256, 4, 4, 64, 1024, False, 300, 1900),
    (768, 12, 12, 64, 3072, False, 20, 2500),    # room for seven of eight shares
    (256, 4, 4, 64, 256, False, 70, 1500),       # MLP rows as wide as the residual stream: planes only, if they hold them
    (512, 2, 2, 128, 2048, False, 257, 0),       # nothing to share
])
def test_shares_stay_inside_the_reported_size(d, hq, hkv, dh, ff, llama, S, pos):
    sh = I.BlockShape(d, hq, hkv, dh, ff, **(dict(norm="rmsnorm", mlp_act="swiglu", use_rope=True, has_bias=False) if llama else {}))
    L, cap = 2, S + pos
    layers = [I.block_weights(sh, 81, l, bf16=True, weight_std=0.05) for l in range(L)]
    tw = [dev_dict(w, True) for w in layers]
    tm = {"normf_g": torch.ones(d, dtype=torch.bfloat16, device="cuda")}
    if not llama:
        tm["normf_b"] = torch.zeros(d, dtype=torch.bfloat16, device="cuda")
    descs = [B.make_block_desc(sh, w) for w in tw]
    model = B.make_model_desc(descs, tm)
    x = I.normal(81, 0, "x", (1, S, d), 1.0, bf16=True)
    kc, vc = (I.normal(81, 0, n, (L, 1, hkv, cap, dh), 1.0, bf16=True) for n in ("k_cache", "v_cache"))

    def guarded(size):      # NaN patterns in the workspace, a guard behind it
        t = torch.full((size + 4096,), 0xff, dtype=torch.uint8, device="cuda")
        return t, t[:size]

    def caches():
        return dev(kc, True), dev(vc, True)

    # one layer against the oracle
    full, ws = guarded(B.forge_decoder_block_workspace_bytes(descs[0], 1, S, cap))
    tk, tv = caches()
    out = torch.empty(1, S, d, dtype=torch.bfloat16, device="cuda")
    B.forge_decoder_block(descs[0], dev(x, True), out, tk[0], tv[0], pos, ws)
    torch.cuda.synchronize()
    k0, v0 = kc[0].astype("float64"), vc[0].astype("float64")
    check(out, O.decoder_block(sh, layers[0], x, k0, v0, pos0=pos), True, "layer behind cached keys", chain=True)
    assert torch.all(full[ws.numel():] == 0xff)

    # the stack, plain and compiled
    full, ws = guarded(B.forge_model_workspace_bytes(model, 1, S, cap))
    k0, v0 = caches()
    plain = torch.empty_like(out)
    B.forge_model_forward(model, dev(x, True), plain, k0, v0, pos, ws)
    torch.cuda.synchronize()
    assert torch.all(full[ws.numel():] == 0xff)
    cm = B.CompiledModel(model, 1, S, pos, cap)
    full, ws = guarded(cm.workspace_bytes())
    k1, v1 = caches()
    got, tx = torch.empty_like(out), dev(x, True)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    cm.bind(tx, got, k1, v1, ws, side)
    side.synchronize()
    for _ in range(2):
        assert torch.equal(got, plain) and torch.equal(k1, k0) and torch.equal(v1, v0)
        got.zero_()
        torch.cuda.synchronize()
        cm.run(side)
        side.synchronize()
    assert torch.equal(got, plain)
    assert torch.all(full[ws.numel():] == 0xff)
    cm.close()
