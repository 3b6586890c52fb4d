"""Performance cases of the framework: what a generation job asks of it on one MI355X.

Three kinds of pass, all through the public binding (`paper_2605_23945_amd.Decoder`):

- "decode":  a batch of requests is admitted with its cached contexts and decoded for `steps` greedy steps, with the
             on-device compaction after each (the protocol of the offline profiler and of the rollout's buckets);
- "prefill": prompts are admitted, their K/V states rebuilt from token ids, the first token decoded, and the states
             handed over as one contiguous buffer (what recomputation yields after a change of the TP layout);
- "switch":  a change of the TP layout on one rank: the old shard's valid K/V gathered, the survivors admitted on the
             new shard, its weights re-sliced from the unsharded layers, its heads filled in, and the first step.

Shapes are the shard shapes of `pat_inputs.CONFIGS`; a smaller depth only repeats the same layer less often.
Contexts are ragged: evenly spread over [ctx / 2, 3 ctx / 2] and shuffled by the seed.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

import paper_2605_23945_amd as pat
import pat_inputs as pi

DEV = "cuda:0"


def listed():
    return [
        # The smallest call: the tiny configuration's 32 greedy steps, where launches and host time are all there is.
        dict(name="decode_tiny_b8", kind="decode", config="tiny_tp1", layers=2, batch=8, ctx=72, steps=32, page=64, qk_norm=False),
        # One sequence left on a narrow shard: the end of a long tail after the switch to a wide TP group.
        dict(name="decode_7b_tp4_b1", kind="decode", config="7b_tp4", layers=32, batch=1, ctx=2047, steps=8, page=64, qk_norm=False),
        # The live batch at which the 7B rollout spends most of its steps.
        dict(name="decode_7b_tp1_b2", kind="decode", config="7b_tp1", layers=32, batch=2, ctx=2900, steps=4, page=64, qk_norm=False),
        # A short tail on the grouped-query shard (one KV head), with the long contexts of its workload.
        dict(name="decode_70b_tp8_b11", kind="decode", config="70b_tp8", layers=40, batch=11, ctx=6001, steps=2, page=64, qk_norm=False),
        # The draining batch on the middle shard, ragged contexts.
        dict(name="decode_13b_tp2_b27", kind="decode", config="13b_tp2", layers=40, batch=27, ctx=1777, steps=1, page=64, qk_norm=False),
        dict(name="decode_7b_tp1_b60", kind="decode", config="7b_tp1", layers=16, batch=60, ctx=1100, steps=1, page=64, qk_norm=False),
        # The model family with per-head q/k normalisation, past the first hundred live sequences.
        dict(name="decode_13b_tp2_b101_qkn", kind="decode", config="13b_tp2", layers=16, batch=101, ctx=1300, steps=1, page=64, qk_norm=True),
        # The start of the 7B rollout: all 256 prompts live, contexts of the prompts and the first tokens.
        dict(name="decode_7b_tp1_b256", kind="decode", config="7b_tp1", layers=8, batch=256, ctx=620, steps=1, page=64, qk_norm=False),
        # A wide live batch on the grouped-query shard.
        dict(name="decode_70b_tp8_b180", kind="decode", config="70b_tp8", layers=20, batch=180, ctx=2100, steps=1, page=64, qk_norm=False),
        # Prompts of the 7B workload prefilled (several of them share a pass of 256 rows).
        dict(name="prefill_7b_tp1_n4", kind="prefill", config="7b_tp1", layers=8, batch=4, ctx=515, width=256, page=64, qk_norm=False),
        # Long contexts rebuilt after a switch on the grouped-query shard, in wide passes.
        dict(name="prefill_70b_tp8_n2", kind="prefill", config="70b_tp8", layers=12, batch=2, ctx=3001, width=1024, page=64, qk_norm=False),
        # A TP change at the tail: 24 survivors, from the unsharded 7B layers to one rank of four.
        dict(name="switch_7b_tp4_n24", kind="switch", config="7b_tp4", layers=8, batch=24, ctx=1501, page=64, qk_norm=False),
    ]


_DEPTH = {"7b_tp1": (4, 16), "7b_tp4": (8, 32), "13b_tp2": (6, 24), "70b_tp8": (8, 40)}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any shard shape, live batch 1..256, contexts 16..8192 (as far as a batch of
    that size is used with them), every page length, both model families."""
    kind = rng.choices(("decode", "prefill", "switch"), weights=(10, 4, 1))[0]
    config = rng.choice(("7b_tp1", "7b_tp4", "13b_tp2", "70b_tp8"))
    page = rng.choice((64, 64, 64, 128, 32, 16))
    lo, hi = _DEPTH[config]
    if kind == "switch":
        batch = _log_int(rng, 2, 40)
        return dict(kind=kind, config=config, layers=rng.randint(2, 5), batch=batch, ctx=_log_int(rng, 100, min(3000, 30000 // batch)),
                    page=page, qk_norm=False)
    qk_norm = rng.random() < 0.2
    if kind == "prefill":
        batch = _log_int(rng, 1, 12)
        tokens = {"7b_tp1": 3500, "7b_tp4": 6000, "13b_tp2": 4000, "70b_tp8": 6000}[config]
        return dict(kind=kind, config=config, layers=rng.randint(2, 8), batch=batch, ctx=_log_int(rng, 40, min(4000, tokens // batch)),
                    width=rng.choice((256, 256, 512, 1024)), page=page, qk_norm=qk_norm)
    batch = _log_int(rng, 1, 256)
    tokens = {"7b_tp1": 80000, "7b_tp4": 160000, "13b_tp2": 120000, "70b_tp8": 400000}[config]      # live context of a batch
    ctx = _log_int(rng, 16, min(8192, tokens // batch))
    steps = max(1, min(8, 16 // batch))
    layers = rng.randint(lo, hi)
    if batch * ctx > tokens // 2:
        layers = min(layers, max(lo, hi // 3))
    return dict(kind=kind, config=config, layers=layers, batch=batch, ctx=ctx, steps=steps, page=page, qk_norm=qk_norm)


# ---- shapes -------------------------------------------------------------------------------------------------

def _shard(case):
    s = pi.CONFIGS[case["config"]]["shard"].with_layers(case["layers"])
    return dataclasses.replace(s, model=dataclasses.replace(s.model, qk_norm=case["qk_norm"]))


def _lens(case):
    """Context lengths of the requests, ascending: batch points spread over [ctx / 2, 3 ctx / 2]."""
    b, ctx = case["batch"], case["ctx"]
    return np.array([max(1, int(ctx * (0.5 + (i + 0.5) / b))) for i in range(b)], np.int64)


def _layer_elems(s):
    return s.hidden * s.qkv_rows + s.hq * s.head_dim * s.hidden + 3 * s.hidden * s.ffn


# ---- inputs -------------------------------------------------------------------------------------------------

def _normal(g, shape, std, mean=0.0):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(mean, std, generator=g)


def _layer(g, s, full=False):
    """One layer's tensors (bf16, N(0, 0.02), gains around 1) of the shard, or of the unsharded model."""
    m, h, d = s.model, s.hidden, s.head_dim
    hq, hkv, f = (m.n_q_heads, m.n_kv_heads, m.ffn) if full else (s.hq, s.hkv, s.ffn)
    w = dict(g1=_normal(g, (h,), 0.02, 1.0), g2=_normal(g, (h,), 0.02, 1.0), wqkv=_normal(g, ((hq + 2 * hkv) * d, h), 0.02),
             wo=_normal(g, (h, hq * d), 0.02), wg=_normal(g, (f, h), 0.02), wu=_normal(g, (f, h), 0.02), wd=_normal(g, (h, f), 0.02))
    if m.qk_norm:
        w.update(gq=_normal(g, (d,), 0.02, 1.0), gk=_normal(g, (d,), 0.02, 1.0))
    return w


def _final(g, s):
    return dict(embed=_normal(g, (s.model.vocab, s.hidden), 0.02), gf=_normal(g, (s.hidden,), 0.02, 1.0),
                wlm=_normal(g, (s.vocab, s.hidden), 0.02))


def _fill_cache(dec, g, s, total):
    """Cached K/V ~ N(0, 1) of all live slots, one layer at a time."""
    slots = list(range(dec.pat_get_state()["live"]))
    for l in range(s.n_layers):
        dec.pat_kv_inject(slots, _normal(g, (1, 2, s.hkv, total, s.head_dim), 1.0), layer0=l)


def prepare(case, seed):
    s, kind = _shard(case), case["kind"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    b, page = case["batch"], case["page"]
    lens = rng.permutation(_lens(case)).astype(np.int32)
    total, steps = int(lens.sum()), case.get("steps", 1)
    target = np.where(np.arange(b) % 8 == 3, steps, steps + 1).astype(np.int32)      # an eighth of a batch finishes with the window
    width = case.get("width", b)
    cfg = pat.make_cfg(s, max(b, width), int(lens.max()) + steps + 1, total + b * (steps + page), page)
    dec = pat.Decoder(cfg, DEV)
    st = dict(kind=kind, dec=dec, steps=steps, ids=np.arange(b, dtype=np.int32), lens=lens, slots=list(range(b)),
              tok=rng.integers(0, s.model.vocab, b, dtype=np.int32), target=target,
              logits=torch.empty(steps, b, s.vocab, device=DEV), next=torch.empty(steps, b, dtype=torch.int32, device=DEV))
    for l in range(s.n_layers):
        dec.pat_load_layer(l, _layer(g, s))
    dec.pat_load_final(_final(g, s))
    dec.pat_decode_admit(st["ids"], st["tok"], lens, st["target"])
    if kind == "prefill":
        st["tokens"] = rng.integers(0, s.model.vocab, total, dtype=np.int32)
    else:
        _fill_cache(dec, g, s, total)
    if kind != "decode":
        st["states"] = torch.empty(s.n_layers, 2, s.hkv, total, s.head_dim, dtype=torch.bfloat16, device=DEV)
    if kind == "switch":        # what the all-gathers of the group return: unsharded layers, the survivors' states of all heads
        st["full"] = [_layer(g, s, full=True) for _ in range(s.n_layers)]
        st["gathered"] = _normal(g, (s.n_layers, 2, s.model.n_kv_heads, total, s.head_dim), 1.0)
        st["head0"] = s.kv_head0
    return st


# ---- one pass -----------------------------------------------------------------------------------------------

def _decode(st):
    dec = st["dec"]
    for i in range(st["steps"]):
        dec.pat_decode_step(False, st["next"][i], st["logits"][i])
        dec.pat_kv_compact()


def run(st):
    dec, kind = st["dec"], st["kind"]
    if kind == "switch":        # the source rank's half
        dec.pat_kv_extract(st["slots"], buf=st["states"])
    dec.pat_decode_reset()
    dec.pat_decode_admit(st["ids"], st["tok"], st["lens"], st["target"])
    if kind == "prefill":
        dec.pat_prefill(st["slots"], st["tokens"])
        dec.pat_kv_extract(st["slots"], buf=st["states"])
    elif kind == "switch":      # the target rank's half
        for l, w in enumerate(st["full"]):
            dec.pat_load_layer_from_full(l, w)
        dec.pat_kv_inject(st["slots"], st["gathered"], n_heads=dec.hkv, buf_head0=st["head0"])
    _decode(st)
    if kind == "switch":        # the next pass finds the source rank's live batch: the slots at their context lengths
        dec.pat_decode_reset()
        dec.pat_decode_admit(st["ids"], st["tok"], st["lens"], st["target"])
    return (st["next"], st["logits"]) if kind == "decode" else (st["next"], st["logits"], st["states"])


# ---- what a pass cannot do without --------------------------------------------------------------------------

def work(case):
    s, lens = _shard(case), _lens(case).astype(float)
    b, nl, d, total = case["batch"], s.n_layers, s.head_dim, float(lens.sum())
    kv_token = 2.0 * s.hkv * d * 2 * nl                       # K and V of one token in all layers
    weights = 2.0 * (nl * _layer_elems(s) + s.vocab * s.hidden)
    steps = case.get("steps", 1)
    mid = total + b * (steps + 1) / 2.0                       # tokens a step attends to, on average
    step_bytes = weights + kv_token * (mid + b) + b * (2.0 * s.hidden + 4.0 * s.vocab)
    step_flops = b * weights + nl * 4.0 * s.hq * d * mid      # two operations per weight and row
    nbytes, flops = steps * step_bytes, steps * step_flops
    if case["kind"] == "prefill":
        nbytes += 2.0 * nl * _layer_elems(s) + total * (2.0 * s.hidden + 3.0 * kv_token)     # written, and read and written again
        flops += 2.0 * nl * _layer_elems(s) * total + nl * 4.0 * s.hq * d * float((lens * (lens + 1) / 2).sum())
    elif case["kind"] == "switch":
        nbytes += 4.0 * kv_token * total + 2 * 2.0 * nl * _layer_elems(s)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Products are good to 2^-17 and sums are fp32; what other summation orders change beyond that is the bf16
    rounding of the appended K/V (an element near a rounding boundary goes the other way), which also moves rebuilt
    states by one bf16 step here and there.  Measured between the kernels of different live batches and pass widths
    on the same rows: rel up to 4.2e-4 (decode) and 6.3e-4 (rebuilt states), max up to 9.3e-3; four times that.
    Tokens may differ where two logits tie within it."""
    return {"rel": 2.5e-3 if case["kind"] == "prefill" else 1.7e-3, "max": 4e-2, "differ": 0.01}
