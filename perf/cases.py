"""The work whose speed is measured, through the public entry points of paper_2604_16498_amd.

A case is a dict of plain values; `listed` gives the fixed ones and `draw` more of the same ranges.
Kinds:
  model      a decoder stack (or, with one layer, a single decoder layer): a prompt of `seq` tokens
             per sequence behind `pos` cached positions, or (`seq` 1) one decode step
  attention  the masked attention operator on its own
Weights are N(0, 0.02), hidden states and cached keys / values N(0, 1), token ids uniform over the
vocabulary, everything drawn on the device from the seed.
"""
import math

import torch

from paper_2604_16498_amd import binding as F
from paper_2604_16498_amd import inputs as I

# layer shape, layers, vocabulary (0: hidden states in and out, no embedding and no head), learned positions.
# Of the large model a stage of 8 of its 32 layers: with all 32 two correct bf16 stacks drift apart
# by more (3 to 4 %) than a comparison of their outputs should allow.
SHAPES = {
    "gpt2s": (I.GPT2_SMALL, 12, 50257, 1024),
    "1p3b": (I.OPT_1P3B, 24, 50272, 2048),
    "8b": (I.LLAMA_8B, 8, 0, 0),
}
_stream = None      # the one side stream of a serving program: its graph replays follow one another


def model(name, shape, batch, seq, pos=0, dtype="bf16", weights="same", ragged=False, replay=False, layer=False):
    """pos: positions already cached (ragged: the largest of them; the sequences then lie evenly
    between a quarter of it and all of it).  weights "int8": per-row quantised.  replay: recorded
    once as a graph, a pass is one replay.  layer: one decoder layer, hidden states in and out."""
    c = {"kind": "model", "shape": shape, "batch": batch, "seq": seq, "pos": pos, "dtype": dtype, "weights": weights,
         "ragged": ragged, "replay": replay, "layer": layer}
    return dict(c, name=name) if name else c


def attention(name, shape, batch, seq):
    c = {"kind": "attention", "shape": shape, "batch": batch, "seq": seq}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small fp32 layer on a 128-token window: full precision, latency and launches count
        model("layer_fp32_b1_s128", "gpt2s", 1, 128, dtype="fp32", layer=True),
        # one 128-token window through the small model: classification, the score of one text
        model("gpt2s_window_b1_s128", "gpt2s", 1, 128),
        # language-model scoring of full contexts, logits of every position
        model("gpt2s_prefill_b8_s1024", "gpt2s", 8, 1024),
        # the generation loop of the small model: one token for 8 sequences of different lengths, the
        # step recorded once as a graph
        model("gpt2s_decode_b8_ragged_replay", "gpt2s", 8, 1, pos=640, ragged=True, replay=True),
        # scoring with the middle model, logits of every position
        model("1p3b_prefill_b4_s2048", "1p3b", 4, 2048),
        # chat serving with the middle model (no shared key / value heads), an odd number of sequences
        model("1p3b_decode_b21_ragged", "1p3b", 21, 1, pos=1400, ragged=True),
        # a long prompt through the large model
        model("8b_prefill_b1_s4096", "8b", 1, 4096),
        # the next turn of a conversation: 777 new tokens behind 2500 cached ones
        model("8b_turn_b1_s777_pos2500", "8b", 1, 777, pos=2500),
        # throughput serving: a full decode batch, contexts of one length
        model("8b_decode_b64_pos2048", "8b", 64, 1, pos=2048),
        # few users with long documents of different lengths
        model("8b_decode_b5_pos8191_ragged", "8b", 5, 1, pos=8191, ragged=True),
        # serving on int8 weights, replayed from a graph
        model("8b_int8_decode_b24_ragged_replay", "8b", 24, 1, pos=1500, weights="int8", ragged=True, replay=True),
        # encoder-style attention over padded texts: every query sees every real key
        attention("masked_attention_b8_s1000", "gpt2s", 8, 1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer_fp32", "gpt2s_prefill", "gpt2s_decode", "1p3b_prefill", "1p3b_decode", "8b_prefill",
                       "8b_decode", "8b_int8_decode", "attention"])
    replay, ragged = rng.random() < 0.5, rng.random() < 0.7
    if kind == "layer_fp32":
        return model("", "gpt2s", rng.randint(1, 4), _log_int(rng, 17, 512), dtype="fp32", layer=True)
    if kind == "gpt2s_prefill":
        return model("", "gpt2s", _log_int(rng, 1, 8), _log_int(rng, 24, 1024), replay=replay)
    if kind == "gpt2s_decode":
        return model("", "gpt2s", _log_int(rng, 1, 64), 1, pos=_log_int(rng, 64, 1000), ragged=ragged, replay=replay)
    if kind == "1p3b_prefill":
        return model("", "1p3b", _log_int(rng, 1, 4), _log_int(rng, 48, 2048), replay=replay)
    if kind == "1p3b_decode":
        return model("", "1p3b", _log_int(rng, 1, 64), 1, pos=_log_int(rng, 96, 2000), ragged=ragged, replay=replay)
    if kind == "8b_prefill":
        seq = _log_int(rng, 80, 4000)
        pos = rng.choice([0, rng.randint(0, 4096 - seq)])
        return model("", "8b", rng.randint(1, max(1, min(3, 4096 // (seq + pos)))), seq, pos=pos, replay=replay)
    if kind == "attention":
        shape = rng.choice(["gpt2s", "1p3b"])
        return attention("", shape, rng.randint(1, 8 if shape == "gpt2s" else 3), _log_int(rng, 100, 1024))
    batch = _log_int(rng, 1, 64)
    pos = _log_int(rng, 128, min(8191, 64 * 2048 // batch))
    return model("", "8b", batch, 1, pos=pos, weights="int8" if kind == "8b_int8_decode" else "same", ragged=ragged,
                 replay=replay)


def _lengths(case):
    """Cached positions of every sequence (in rising order)."""
    b, top = case["batch"], case["pos"]
    if not case["ragged"]:
        return [top] * b
    return [top - (3 * top * (b - 1 - i)) // (4 * max(1, b - 1)) for i in range(b)]


def _layers(case):
    return 1 if case["layer"] else SHAPES[case["shape"]][1]


def _vocab(case):
    return 0 if case["layer"] else SHAPES[case["shape"]][2]


def _weights(sh, int8, dt, normal):
    """One layer's tensors under the names of the block descriptor."""
    d = sh.d_model
    w = {"norm1_g": 1.0 + normal((d,), 0.1), "norm2_g": 1.0 + normal((d,), 0.1)}
    if sh.norm == "layernorm":
        w.update(norm1_b=normal((d,), 0.1), norm2_b=normal((d,), 0.1))
    for name, n, k in (("qkv", sh.qkv_out, d), ("o", d, sh.q_heads * sh.head_dim), ("up", sh.up_out, d),
                       ("down", d, sh.d_ff)):
        w["w_" + name] = normal((n, k), 0.02)
        if int8:
            w["w_" + name], w["s_" + name] = F.forge_quantize_int8(w["w_" + name])
        if sh.has_bias:
            w["b_" + name] = normal((n,), 0.02)
    return w


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if case.get("dtype") == "fp32" else torch.bfloat16
    sh, _, _, n_pos = SHAPES[case["shape"]]
    B, S = case["batch"], case["seq"]

    def normal(shape, std=1.0):
        return torch.randn(shape, generator=g, device="cuda", dtype=dt).mul_(std)

    if case["kind"] == "attention":
        # padded texts: of every sequence the keys from its length on are cut
        lengths = torch.randint(max(1, S // 2), S + 1, (B,), generator=g, device="cuda")
        keys = torch.arange(S, device="cuda")
        mask = torch.where(keys[None, :] < lengths[:, None], 0.0, -torch.inf)
        mask = mask[:, None, None, :].expand(B, 1, S, S).contiguous()
        q = normal((B, sh.q_heads, S, sh.head_dim))
        k, v = (normal((B, sh.kv_heads, S, sh.head_dim)) for _ in range(2))
        return {"case": case, "q": q, "k": k, "v": v, "mask": mask,
                "out": torch.zeros(B, S, sh.q_heads * sh.head_dim, device="cuda", dtype=dt)}

    layers, vocab, pos = _layers(case), _vocab(case), case["pos"]
    weights = [_weights(sh, case["weights"] == "int8", dt, normal) for _ in range(layers)]
    descs = [F.make_block_desc(sh, w) for w in weights]
    cap = (pos + S + 63) // 64 * 64
    kc, vc = (torch.zeros(layers, B, sh.kv_heads, cap, sh.head_dim, device="cuda", dtype=dt) for _ in range(2))
    if pos:
        for cache in (kc, vc):
            for i in range(layers):
                cache[i, :, :, :pos] = normal((B, sh.kv_heads, pos, sh.head_dim))
    st = {"case": case, "weights": weights, "descs": descs, "kc": kc, "vc": vc}
    if case["ragged"]:
        order = torch.randperm(B, generator=g, device="cuda")
        st["seq_pos"] = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")[order].contiguous()
    if case["layer"]:
        st["inp"] = normal((B, S, sh.d_model))
        st["out"] = torch.zeros_like(st["inp"])
        st["ws"] = F.workspace(F.forge_decoder_block_workspace_bytes(descs[0], B, S, cap))
        st["kc"], st["vc"] = kc[0], vc[0]
        return st
    mw = {"normf_g": 1.0 + normal((sh.d_model,), 0.1)}
    if sh.norm == "layernorm":
        mw["normf_b"] = normal((sh.d_model,), 0.1)
    ld = (vocab + 7) // 8 * 8            # logits rows padded to 16 bytes
    if vocab:
        mw.update(wte=normal((vocab, sh.d_model), 0.02), wpe=normal((n_pos, sh.d_model), 0.02))
        st["inp"] = torch.randint(0, vocab, (B, S), generator=g, device="cuda", dtype=torch.int32)
    else:
        st["inp"] = normal((B, S, sh.d_model))
    st["out"] = torch.zeros(B, S, ld if vocab else sh.d_model, device="cuda", dtype=dt)
    st["mw"] = mw
    st["model"] = F.make_model_desc(descs, mw, logits_ld=ld)
    if not case["replay"]:
        st["ws"] = F.workspace(F.forge_model_workspace_bytes(st["model"], B, S, cap))
        return st
    st["compiled"] = F.CompiledModel(st["model"], B, S, pos, cap)
    st["ws"] = F.workspace(st["compiled"].workspace_bytes())
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    st["stream"] = _stream
    _stream.wait_stream(torch.cuda.current_stream())
    if case["ragged"]:
        st["compiled"].bind_decode(st["inp"], st["out"], kc, vc, st["seq_pos"], st["ws"], st["stream"])
    else:
        st["compiled"].bind(st["inp"], st["out"], kc, vc, st["ws"], st["stream"])
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "attention":
        return F.forge_attn_fused_masked(st["q"], st["k"], st["v"], st["mask"], st["out"], causal=False)
    out, kc, vc, pos = st["out"], st["kc"], st["vc"], case["pos"]
    if case["layer"]:
        F.forge_decoder_block(st["descs"][0], st["inp"], out, kc, vc, pos, st["ws"])
    elif case["replay"]:
        st["compiled"].run(st["stream"])
    elif case["ragged"]:
        F.forge_model_decode(st["model"], st["inp"], out, kc, vc, st["seq_pos"], pos, st["ws"])
    else:
        F.forge_model_forward(st["model"], st["inp"], out, kc, vc, pos, st["ws"])
    return {"out": out, "k_cache": kc, "v_cache": vc}


def work(case):
    sh = SHAPES[case["shape"]][0]
    es = 4 if case.get("dtype") == "fp32" else 2
    B, S, hd = case["batch"], case["seq"], sh.q_heads * sh.head_dim
    if case["kind"] == "attention":
        return {"bytes": B * S * (2 * hd + 2 * sh.kv_heads * sh.head_dim) * es + 4.0 * B * S * S,
                "flops": 4.0 * B * sh.q_heads * S * S * sh.head_dim}
    layers, vocab = _layers(case), _vocab(case)
    n_w = sh.d_model * (sh.qkv_out + hd + sh.up_out + sh.d_ff)
    kv_row = 2 * sh.kv_heads * sh.head_dim
    pairs = sum(p * S + S * (S + 1) // 2 for p in _lengths(case))     # (query, key) pairs of a head
    flops = layers * (2.0 * B * S * n_w + 4.0 * hd * pairs) + 2.0 * B * S * sh.d_model * vocab
    w_bytes = n_w * (1 if case["weights"] == "int8" else es)
    kv_bytes = (sum(_lengths(case)) + B * S) * kv_row * es            # cached rows read, new rows written
    ends = B * S * ((4 + 2 * sh.d_model * es if vocab else sh.d_model * es) + (vocab or sh.d_model) * es)
    return {"bytes": float(layers * (w_bytes + kv_bytes) + vocab * sh.d_model * es + ends), "flops": flops}


def tolerance(case):
    """About four times what the outputs and the new cache rows differ by from the same stack in fp32
    (the fp32 layer: from fp64) on the same inputs, and never over 3 %."""
    if case.get("dtype") == "fp32":
        return {"rel": 2e-6, "max": 2e-5}         # measured 3e-7, 2e-6
    if case["kind"] == "attention":
        return {"rel": 9e-3, "max": 5e-2}         # measured 2.2e-3, 1.1e-2
    return {"rel": 3e-2, "max": 0.3}              # measured 0.8 to 1.4e-2, 0.03 to 0.09
