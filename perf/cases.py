"""The performance cases of the coded-KV path: what a serving program asks of this library.

A case is a dict of plain values.  `op` names the call a pass makes through the public entry points:
  decode    one decode step of attention over the coded cache of `layers` layers (each layer has a cache of
            its own, as in a model), with or without the fp16 residual rows
  encode    prefill of whole prompts, or the flush of a full 64-token residual, of `layers` layers
  step      a decode step that encodes its one new token per sequence first and then attends
  codebook  K-Means codebook on normal samples, followed by cosine fine-tuning where asked
Code formats: sub_dim 4 = 2-bit, sub_dim 8 = 1-bit, sign = the 2-bit format with sign bytes; rope = keys
normalised before the rotary embedding; side_bits 4 = double quantization; group = tokens per Shift mean.
Lengths are uniform in [len_lo, len_hi], drawn with len_seed (they are part of the case, not of the inputs).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_18231_amd import api, synth

D = 128
RES = 64                 # rows of the fp16 residual
SCALE = 1.0 / math.sqrt(D)
ROPE_BASE = 500000.0
FINETUNE_LR = 2048.0

_ATTN = dict(layers=1, batch=1, q_heads=32, kv_heads=8, len_lo=1024, len_hi=1024, len_seed=0, sub_dim=4, sign=False,
             rope=False, side_bits=16, group=0, page=0)


def _decode(**kw):
    return dict(_ATTN, op="decode", residual=False, **kw)


def _encode(**kw):
    return dict(_ATTN, op="encode", flush=False, **kw)


def listed():
    cases = [
        # one short conversation on one head pair: the smallest call, where only latency counts
        dict(_decode(), name="decode_tiny_1bit", q_heads=1, kv_heads=1, len_lo=1024, len_hi=1024, sub_dim=8),
        # the ordinary decode step of a grouped-query model, 8 sequences of 8192 tokens, residual partly filled
        dict(_decode(), name="decode_gqa_2bit_residual", layers=4, batch=8, len_lo=8192, len_hi=8192, residual=True),
        # one very long context, 1-bit: the token axis has to be split to fill the chip
        dict(_decode(), name="decode_long_context_1bit", layers=4, len_lo=131072, len_hi=131072, sub_dim=8),
        # continuous batching: 32 requests of very different lengths in a paged cache
        dict(_decode(), name="decode_ragged_paged_2bit", layers=2, batch=32, len_lo=512, len_hi=16384, len_seed=4,
             page=256),
        # throughput serving of a multi-head model: the largest cache, bound by HBM
        dict(_decode(), name="decode_mha_large_2bit", batch=64, q_heads=32, kv_heads=32, len_lo=32768, len_hi=32768),
        # the method with all of the paper's options (sign + index codes, 64-token groups, keys before the rotary
        # embedding, double quantization, residual) on the ordinary shape
        dict(_decode(), name="decode_paper_format", layers=4, batch=8, len_lo=8192, len_hi=8192, sub_dim=8, sign=True,
             rope=True, side_bits=4, group=64, residual=True),
        # the paper's 2-bit codes with fp16 side information, requests of different lengths in pages
        dict(_decode(), name="decode_sign_ragged_paged", layers=2, batch=16, len_lo=512, len_hi=8192, len_seed=7,
             sub_dim=8, sign=True, group=64, page=256, residual=True),
        # prefill of eight long prompts, 2-bit
        dict(_encode(), name="encode_prefill_2bit", batch=8, len_lo=8192, len_hi=8192),
        # prefill with all of the paper's options, 4 prompts of up to 4096 tokens (odd lengths)
        dict(_encode(), name="encode_prefill_paper", batch=4, len_lo=2048, len_hi=4096, len_seed=9, sub_dim=8, sign=True,
             rope=True, side_bits=4, group=64),
        # every 64th step of a decode loop: the full residual of 8 sequences goes into the cache
        dict(_encode(), name="encode_residual_flush", layers=4, batch=8, len_lo=8192, len_hi=8192, flush=True),
        # a decode step without a residual: 32 ragged sequences append one token each, then attend, 1-bit
        dict(_ATTN, op="step", name="step_append_paged_1bit", layers=2, batch=32, len_lo=512, len_hi=16384, len_seed=4,
             sub_dim=8, page=256),
        # the magnitude codebook of the paper's format: K-Means, then cosine fine-tuning
        dict(op="codebook", name="codebook_build_finetune", sub_dim=8, sign=True, samples=1 << 20, iters=50,
             finetune_iters=20),
    ]
    return cases


# ---- more cases of the same ranges -----------------------------------------------------------------
MAX_DECODE_UNITS = 64 * 32 * 32768       # tokens x kv heads x layers of the largest listed decode
MAX_ENCODE_UNITS = 8 * 8 * 8192          # of the largest listed prefill


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_format(rng, case):
    kind = rng.choice(("2bit", "2bit", "1bit", "1bit", "sign", "sign"))
    case["sub_dim"] = 4 if kind == "2bit" else 8
    case["sign"] = kind == "sign"
    case["rope"] = rng.random() < 0.25
    case["side_bits"] = 4 if rng.random() < 0.25 else 16
    case["group"] = rng.choice((0, 64)) if kind != "sign" else rng.choice((0, 64, 64))
    case["page"] = rng.choice((0, 0, 64, 256))


def _draw_heads(rng, case):
    case["kv_heads"] = rng.choice((1, 2, 4, 8, 8, 16, 32))
    case["q_heads"] = case["kv_heads"] * rng.choice([r for r in (1, 2, 3, 4, 4, 6, 8) if r * case["kv_heads"] <= 64])


def _draw_lengths(rng, case, longest):
    hi = _log_int(rng, 65, max(66, longest))
    lo = hi if rng.random() < 0.4 else max(1, int(hi * rng.uniform(0.03, 0.9)))
    case.update(len_lo=lo, len_hi=hi, len_seed=rng.randrange(1 << 20))


def draw(rng):
    kind = rng.random()
    if kind < 0.1:
        sub = rng.choice((4, 8))
        n = _log_int(rng, 1 << 13, 1 << 20)
        return dict(op="codebook", sub_dim=sub, sign=sub == 8 and rng.random() < 0.5, samples=n, iters=rng.randint(5, 50),
                    finetune_iters=rng.choice((0, rng.randint(1, 20))))
    if kind < 0.6:
        case = _decode()
    elif kind < 0.9:
        case = _encode()
    else:
        case = dict(_ATTN, op="step")
    _draw_format(rng, case)
    _draw_heads(rng, case)
    case["batch"] = _log_int(rng, 1, 64)
    case["layers"] = rng.choice((1, 2, 4))
    per_token = case["batch"] * case["kv_heads"] * case["layers"]
    if case["op"] == "encode":
        case["flush"] = rng.random() < 0.35
        limit = MAX_ENCODE_UNITS // per_token
        if case["flush"]:
            while case["batch"] * case["kv_heads"] * case["layers"] * RES > MAX_ENCODE_UNITS:
                case["batch"] //= 2
            _draw_lengths(rng, case, 8192)
        else:
            while limit < 256:
                case["batch"] = max(1, case["batch"] // 2)
                limit = MAX_ENCODE_UNITS // (case["batch"] * case["kv_heads"] * case["layers"])
            _draw_lengths(rng, case, min(16384, limit))
    else:
        _draw_lengths(rng, case, min(131072, max(256, MAX_DECODE_UNITS // 2 // per_token)))
        if case["op"] == "decode":
            case["residual"] = rng.random() < 0.5
        else:                      # single-token appends use the stored mean of the sequence
            case.update(side_bits=16, group=0)
    return case


# ---- inputs ----------------------------------------------------------------------------------------
def _lengths(case):
    g = np.random.RandomState(case["len_seed"])
    n = g.randint(case["len_lo"], case["len_hi"] + 1, size=case["batch"]).astype(np.int64)
    if case.get("residual") or case.get("flush"):   # whole residuals have been encoded so far
        n = n // RES * RES
        n[:] = np.maximum(n, RES)
    return n


def _residual_lengths(case):
    return np.random.RandomState(case["len_seed"] + 1).randint(0, RES + 1, size=case["batch"])


def _room(case):
    unit = max(RES, case["page"])
    return int((_lengths(case).max() + RES + unit - 1) // unit * unit)


def _bytes_per_token(case):
    return 32 if case["sign"] else D // case["sub_dim"]


def _keys(gen, stats, batch, n):
    x = torch.randn((batch, stats[0].shape[0], n, D), generator=gen, device="cuda", dtype=torch.float16)
    return x.mul_(stats[0]).add_(stats[1])


def _values(gen, batch, heads, n):
    return torch.randn((batch, heads, n, D), generator=gen, device="cuda", dtype=torch.float16)


def _channel_stats(gen, heads):
    """Per-channel scale and bias of keys: log-normal scales, wide biases, two outlier channels per head."""
    scale = torch.exp(torch.randn((heads, 1, D), generator=gen, device="cuda"))
    bias = 2.0 * torch.randn((heads, 1, D), generator=gen, device="cuda")
    order = torch.rand((heads, 1, D), generator=gen, device="cuda").argsort(dim=-1)
    bias += 20.0 * (order < 2)
    return scale.half(), bias.half()


def _samples(case, seed, n):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((n, case["sub_dim"]), generator=gen, device="cuda")
    return x.abs() if case["sign"] else x


def _codebook(case, seed):
    cb, _ = api.nsn_build_codebook(_samples(case, seed, 1 << 15), 256, 8)
    if case["side_bits"] == 4:
        api.nsn_quantize_codebook(cb)
    return cb


def prepare(case, seed):
    if case["op"] == "codebook":
        ws = api.nsn_workspace_bytes(api.make_shape(case["sub_dim"], 1, 1, 64), api.NSN_OP_CODEBOOK, 1, case["samples"])
        return dict(case=case, samples=_samples(case, seed, case["samples"]),
                    workspace=torch.empty(ws, dtype=torch.uint8, device="cuda"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, Hq, Hkv = case["batch"], case["q_heads"], case["kv_heads"]
    room, lens = _room(case), _lengths(case)
    rope = api.nsn_build_rope_table(synth.rope_inv_freq(ROPE_BASE), room) if case["rope"] else None
    shape = api.make_shape(case["sub_dim"], Hq, Hkv, room, case["group"], case["page"], sign_format=case["sign"],
                           rope_table=rope, side_bits=case["side_bits"])
    cb = _codebook(case, seed)
    table = None
    if case["page"]:
        pages = B * (room // case["page"])
        table = torch.randperm(pages, generator=gen, device="cuda").to(torch.int32).view(B, room // case["page"])
    lens_d = torch.tensor(lens, dtype=torch.int32, device="cuda")
    state = dict(case=case, shape=shape, codebook=cb, lens=lens_d, longest=int(lens.max()), layers=[])
    encode_only = case["op"] == "encode" and not case["flush"]
    longest = int(lens.max())
    for _ in range(case["layers"]):
        layer = dict(k_cache=api.alloc_cache(shape, B, block_table=table), v_cache=api.alloc_cache(shape, B, block_table=table))
        stats = _channel_stats(gen, Hkv)
        if encode_only:
            layer["k"], layer["v"] = _keys(gen, stats, B, longest), _values(gen, B, Hkv, longest)
        else:                      # the tokens cached so far: some sequences at a time, as prompts arrive
            n_seq = max(1, min(B, (1 << 29) // (Hkv * longest * D)))
            for b in range(0, B, n_seq):
                some = slice(b, min(b + n_seq, B))
                n = int(lens[some].max())
                part = [_sequences(layer[c], some) for c in ("k_cache", "v_cache")]
                api.nsn_encode(shape, cb, _keys(gen, stats, some.stop - b, n), _values(gen, some.stop - b, Hkv, n),
                               torch.zeros(some.stop - b, dtype=torch.int32, device="cuda"), lens_d[some], *part)
            new = RES if case.get("flush") or case.get("residual") else 1
            layer["k"], layer["v"] = _keys(gen, stats, B, new), _values(gen, B, Hkv, new)
        layer["q"] = torch.randn((B, Hq, D), generator=gen, device="cuda", dtype=torch.float16)
        layer["out"] = torch.empty((B, Hq, D), dtype=torch.float32, device="cuda")
        state["layers"].append(layer)
    if case["op"] == "encode":
        state["start"] = lens_d if case["flush"] else torch.zeros(B, dtype=torch.int32, device="cuda")
        state["n_new"] = torch.full((B,), RES, dtype=torch.int32, device="cuda") if case["flush"] else lens_d
        state["freeze"] = case["flush"] and case["group"] == 0
    elif case["op"] == "step":
        state["n_new"] = torch.ones(B, dtype=torch.int32, device="cuda")
        state["lens_after"] = lens_d + 1
    elif case["residual"]:
        state["res_lens"] = torch.tensor(_residual_lengths(case), dtype=torch.int32, device="cuda")
    n_new = state["layers"][0]["k"].shape[2]
    if case["op"] in ("encode", "step"):
        need = api.nsn_workspace_bytes(shape, api.NSN_OP_ENCODE, B, n_new)
        state["encode_ws"] = torch.empty(max(1, need), dtype=torch.uint8, device="cuda")
    if case["op"] in ("decode", "step"):
        need = api.nsn_workspace_bytes(shape, api.NSN_OP_DECODE, B)
        state["decode_ws"] = torch.zeros(max(1, need), dtype=torch.uint8, device="cuda")
    return state


def _sequences(cache, some):
    """The cache of some of the sequences (pages are shared, everything else is per sequence)."""
    if cache.block_table is not None:
        return api.CodedCache(cache.codes, cache.norms, cache.means[some], cache.block_table[some])
    return api.CodedCache(cache.codes[some], cache.norms[some], cache.means[some], None)


# ---- one pass --------------------------------------------------------------------------------------
def _encode_layer(s, layer, start, freeze):
    api.nsn_encode(s["shape"], s["codebook"], layer["k"], layer["v"], start, s["n_new"], layer["k_cache"], layer["v_cache"],
                   freeze_means=freeze, workspace=s["encode_ws"])


def _cache_tensors(layer):
    return [t for c in (layer["k_cache"], layer["v_cache"]) for t in (c.codes, c.norms, c.means)]


def run(state):
    s, case = state, state["case"]
    if case["op"] == "codebook":
        cb, mse = api.nsn_build_codebook(s["samples"], 256, case["iters"], workspace=s["workspace"])
        if not case["finetune_iters"]:
            return cb, mse
        return (mse,) + tuple(api.nsn_finetune_codebook(s["samples"], cb, case["finetune_iters"], FINETUNE_LR,
                                                        workspace=s["workspace"]))
    outs = []
    for layer in s["layers"]:
        if case["op"] == "encode":
            _encode_layer(s, layer, s["start"], s["freeze"])
            outs += _cache_tensors(layer)
            continue
        if case["op"] == "step":
            _encode_layer(s, layer, s["lens"], True)
            api.nsn_decode_attention(s["shape"], s["codebook"], layer["q"], layer["k_cache"], layer["v_cache"],
                                     s["lens_after"], s["longest"] + 1, SCALE, out=layer["out"], workspace=s["decode_ws"])
            outs += _cache_tensors(layer)
        elif case["residual"]:
            api.nsn_decode_attention_residual(s["shape"], s["codebook"], layer["q"], layer["k_cache"], layer["v_cache"],
                                              s["lens"], s["longest"], layer["k"], layer["v"], s["res_lens"], SCALE,
                                              out=layer["out"], workspace=s["decode_ws"])
        else:
            api.nsn_decode_attention(s["shape"], s["codebook"], layer["q"], layer["k_cache"], layer["v_cache"], s["lens"],
                                     s["longest"], SCALE, out=layer["out"], workspace=s["decode_ws"])
        outs.append(layer["out"])
    return outs


# ---- what a pass cannot do without -------------------------------------------------------------------
def _coded_bytes(case, lens):
    """Cache bytes (K and V) of sequences of these lengths: codes, token scales, means."""
    tokens, dq = int(lens.sum()), case["side_bits"] == 4
    groups = int(((lens + case["group"] - 1) // case["group"]).sum()) if case["group"] else len(lens)
    per_token = 2 * _bytes_per_token(case) + (2 * 164 / 64 if dq else 8)
    return case["kv_heads"] * (tokens * per_token + groups * 2 * (80 if dq else 2 * D))


def work(case):
    if case["op"] == "codebook":
        passes = case["iters"] + 1 + (case["finetune_iters"] + 2 if case["finetune_iters"] else 0)
        return dict(bytes=case["samples"] * case["sub_dim"] * 4 + 256 * case["sub_dim"] * 2,
                    flops=passes * case["samples"] * 256 * 2 * case["sub_dim"])
    lens, B, Hq, Hkv = _lengths(case), case["batch"], case["q_heads"], case["kv_heads"]
    codebook = 256 * case["sub_dim"] * 2
    new_bytes = new_flops = attn_bytes = attn_flops = 0
    if case["op"] != "decode":                      # tokens encoded by this pass
        new = lens if case["op"] == "encode" and not case["flush"] else np.full(B, RES if case["op"] == "encode" else 1)
        n = int(new.sum()) * Hkv * 2
        new_bytes = n * D * 2 + _coded_bytes(case, new) + codebook
        new_flops = n * (D * 256 * 2 + D * 7 * 2 + 12 * D)  # codeword distances, rotation, two Normalize and a Shift
    if case["op"] != "encode":
        rows = int(_residual_lengths(case).sum()) if case.get("residual") else 0
        attn_bytes = _coded_bytes(case, lens) + rows * Hkv * 2 * D * 2 + B * Hq * D * (2 + 4) + codebook
        attn_flops = (int(lens.sum()) + rows) * Hq * 4 * D
    return dict(bytes=int(case["layers"] * (new_bytes + attn_bytes)), flops=int(case["layers"] * (new_flops + attn_flops)))


def tolerance(case):
    if case["op"] == "codebook":
        return dict(rel=1e-4, max=2e-3)             # fp16 entries rounded once from fp64 sums: a unit in a few of them
    if case["op"] == "encode":
        return dict(rel=1e-4, max=2e-3, differ=1e-5)  # fp16 scales rounded once; codewords at equal distance (1e-6)
    return dict(rel=2e-3, max=2e-2, differ=1e-5)    # the softmax weights meet the values as fp16
