"""Parity of the prefill (recomputation) path against the CPU oracle: K/V of every position and
layer within one bf16 step, the decode steps that follow within the logit tolerance with identical
tokens, slots not named left byte-identical, error paths."""
import numpy as np
import pytest
import torch

import pat_inputs as pi
from gpu_util import DEV, bf16_close, check_logits, make_decoder, make_oracle_decoder, oracle_admit
from oracle import bits, prefill

pytestmark = pytest.mark.gpu


def _pat():
    import paper_2605_23945_amd as p
    return p


def _kv_bits(dec, slot, n_layers, L):
    out = []
    for l in range(n_layers):
        if L == 0:
            out.append((np.zeros(0, np.uint16), np.zeros(0, np.uint16)))
            continue
        k, v = dec.pat_kv_read(slot, l, L)
        out.append((bits(k.cpu()), bits(v.cpu())))
    return out


def _prefill_parity(shard, kv_lens, slots, max_batch, page_tokens=64, steps=2, chunked=None, chunk=None):
    pat = _pat()
    n = len(kv_lens)
    req = pi.rollout_requests(shard, n, (1, 2), steps=steps + 1)
    req["kv_len"] = np.asarray(kv_lens, np.int32)
    dec = make_decoder(shard, max_batch, int(max(kv_lens)) + steps + 2, int(sum(kv_lens)) + (steps + 64) * n, page_tokens)
    pat.admit_synthetic(dec, shard, req, DEV)
    odec = make_oracle_decoder(shard)
    oracle_admit(odec, shard, req, range(n), steps + 2)
    before = [_kv_bits(dec, j, shard.n_layers, int(kv_lens[j])) for j in range(n)]
    toks = [pi.prompt_tokens(shard, int(req["seq_id"][j]), int(kv_lens[j])) for j in slots]
    print(f"prefill: slots {list(slots)}, lengths {[int(kv_lens[j]) for j in slots]}, pass width {max_batch}", flush=True)
    dec.pat_prefill(slots, np.concatenate(toks) if toks else np.zeros(0, np.int32))
    if chunked is not None:
        assert (dec.pat_attention_cut()["prefill"][1] > 0) == chunked
    assert chunk is None or dec.pat_attention_cut()["prefill"][0] == chunk
    for j, t in zip(slots, toks):
        prefill(odec, j, t)
    st = dec.pat_get_state()
    assert np.array_equal(st["kv_len"], req["kv_len"]) and np.all(st["gen"] == 0) and np.array_equal(st["token"], req["token"])
    for j in range(n):
        L = int(kv_lens[j])
        got = _kv_bits(dec, j, shard.n_layers, L)
        for l in range(shard.n_layers):
            if j not in slots:                                   # not named: untouched, byte for byte
                assert np.array_equal(got[l][0], before[j][l][0]) and np.array_equal(got[l][1], before[j][l][1])
                continue
            if L == 0:
                continue
            for g, ref in ((got[l][0], odec.kc[j][l][:L]), (got[l][1], odec.vc[j][l][:L])):
                # Every element within one bf16 step.  Layer 0 sees exact inputs: its fp32 k, v are good
                # to ~1e-5 of their scale, so only ~0.3 % of the elements sit close enough to a rounding
                # boundary to round the other way.  A deeper layer's input carries those flipped elements
                # (each off by 2^-8 of itself) of this and the earlier positions: they move the residual,
                # and with it the next layer's k, v before rounding, by 1e-4 .. 6e-4 (rms over a
                # position's features) of the tensor's scale, which flips ~10 % of its elements; over the
                # 4096 features of a position the largest such deviation is ~3.5 sigma = 2e-3, so 4e-3 of
                # the tensor's rms is allowed on top of the bf16 step there.
                same, close = bf16_close(g, ref, abs_tol=5e-4 if l == 0 else 4e-3)
                assert close and same > (0.97 if l == 0 else 0.85), (j, l, same, close)
    worst = 0.0
    for _ in range(steps):                                       # the decode steps run from the rebuilt states
        ref_logits, ref_next, _ = odec.step()
        logits = torch.empty(n, shard.vocab, device=DEV); nxt = torch.empty(n, dtype=torch.int32, device=DEV)
        dec.pat_decode_step(True, nxt, logits)
        worst = max(worst, check_logits(logits.cpu().numpy(), ref_logits))
        assert np.array_equal(nxt.cpu().numpy(), ref_next)
    dec.close()
    return worst


def test_tiny_ragged_sequences_in_one_pass():
    """Lengths 0, 1, one short of / on / past a page boundary; rows of all sequences share one pass."""
    shard = pi.CONFIGS["tiny_tp1"]["shard"]
    _prefill_parity(shard, [0, 1, 15, 16, 17, 90], [0, 1, 2, 3, 4, 5], max_batch=256, page_tokens=16)


def test_tiny_many_passes_and_a_subset_of_slots_in_any_order():
    """Pass width 4: a sequence spans many passes and attends to rows of earlier passes; only slots
    3 and 1 are rebuilt (in that order), the rest keep their states."""
    shard = pi.CONFIGS["tiny_tp1"]["shard"]
    _prefill_parity(shard, [9, 30, 5, 21], [3, 1], max_batch=4, page_tokens=16)


def test_tiny_long_sequence_spanning_passes():
    """300 + 270 positions at pass width 256: three passes."""
    shard = pi.CONFIGS["tiny_tp1"]["shard"]
    _prefill_parity(shard, [300, 270], [0, 1], max_batch=256)


@pytest.mark.parametrize("lens,width", [((200, 150, 90), 320), ((300, 200, 30), 530), ((500, 400, 124), 1000)])
def test_pass_wider_than_one_projection_group(lens, width):
    """Passes of 320, 530 and 1000 rows: three to sixteen row groups in a projection's launch, the last one ragged."""
    shard = pi.CONFIGS["tiny_tp1"]["shard"]
    _prefill_parity(shard, list(lens), [0, 1, 2], max_batch=width, page_tokens=16)


@pytest.mark.parametrize("tp,rank", [(2, 1)])
def test_tp_shard_prefill(tp, rank):
    shard = pi.ShardShape(pi.CONFIGS["tiny_tp1"]["shard"].model, tp, rank)
    _prefill_parity(shard, [40, 7], [0, 1], max_batch=64, page_tokens=16)


def test_grouped_query_prefill():
    import dataclasses
    base = pi.CONFIGS["tiny_tp1"]["shard"]
    shard = pi.ShardShape(dataclasses.replace(base.model, n_q_heads=8, n_kv_heads=2, head_dim=64), 1, 0)
    _prefill_parity(shard, [70, 33], [0, 1], max_batch=128)


def test_per_head_qk_norm_prefill():
    import dataclasses
    base = pi.CONFIGS["tiny_tp1"]["shard"]
    shard = pi.ShardShape(dataclasses.replace(base.model, qk_norm=True), 1, 0)
    _prefill_parity(shard, [50, 20], [1, 0], max_batch=48, page_tokens=16)


def test_7b_shape_two_layers_prefill_spanning_two_passes():
    """The headline model's layer shape: 200 + 70 rows, 256 in the first pass (the full-batch
    projection kernels), 14 in the second."""
    shard = pi.CONFIGS["7b_tp1"]["shard"].with_layers(2)
    _prefill_parity(shard, [200, 70], [0, 1], max_batch=256, steps=1)


def test_error_paths_change_nothing():
    pat = _pat()
    shard = pi.CONFIGS["tiny_tp1"]["shard"]
    req = pi.rollout_requests(shard, 3, (5, 9), steps=2)
    dec = make_decoder(shard, 4, 32, 200, 16)
    pat.admit_synthetic(dec, shard, req, DEV)
    L = req["kv_len"]
    before = [_kv_bits(dec, j, shard.n_layers, int(L[j])) for j in range(3)]
    ok = np.zeros(int(L[0]), np.int32)
    for slots, toks, code in (([0], np.zeros(int(L[0]) + 1, np.int32), pat.binding.PAT_EINVAL),       # count mismatch
                              ([3], ok, pat.binding.PAT_EINVAL),                                       # not live
                              ([0, 0], np.zeros(2 * int(L[0]), np.int32), pat.binding.PAT_EINVAL),     # repeated
                              ([0], np.full(int(L[0]), shard.model.vocab, np.int32), pat.binding.PAT_EINVAL),
                              ([0], np.full(int(L[0]), -1, np.int32), pat.binding.PAT_EINVAL)):
        with pytest.raises(pat.PatError) as e:
            dec.pat_prefill(slots, toks)
        assert e.value.code == code
    for j in range(3):
        got = _kv_bits(dec, j, shard.n_layers, int(L[j]))
        for l in range(shard.n_layers):
            assert np.array_equal(got[l][0], before[j][l][0]) and np.array_equal(got[l][1], before[j][l][1])
    dec.close()


def test_profile_prefill_table_feeds_the_switch_decision():
    """The prefill half of the offline profiler: row order, skipped points, a latency that grows with the
    work, an empty batch afterwards; the rows serve as the T_prefill table of the switch decision, whose
    recomputation cost then equals the profiled latency at a profiled point."""
    pat = _pat()
    shard = pi.CONFIGS["tiny_tp1"]["shard"]
    dec = make_decoder(shard, 64, 600, 8 * 600 + 64 * 64, 16)
    arr, rows = dec.pat_profile_prefill([1, 4, 8], [64, 512, 1024], 4 * 512, reps=2)
    assert [(r["batch"], r["length"]) for r in rows] == [(b, L) for b in (1, 4, 8) for L in (64, 512, 1024)]
    assert all(r["tp_degree"] == 1 for r in rows)
    lat = {(r["batch"], r["length"]): r["latency_us"] for r in rows}
    assert lat[(8, 512)] == -1.0                    # 8 * 512 tokens exceed the token cap
    assert all(lat[(b, 1024)] == -1.0 for b in (1, 4, 8))   # longer than max_seq_len
    for key in ((1, 64), (1, 512), (4, 64), (4, 512), (8, 64)):
        assert lat[key] > 0.0
    assert lat[(4, 512)] > lat[(4, 64)] and lat[(4, 512)] > lat[(1, 512)]
    assert dec.pat_get_state()["live"] == 0 and len(dec.pat_get_pages()[1]) == dec.req.n_pages
    dec.close()
    # Algorithm 1 with this table: four unfinished samples of length 512 restored on one TP=1 group of a
    # one-GPU "node"; recomputation is looked up at the profiled point (batch 4, length 512) itself
    grid = [(tp, b, T, 1000.0 + 0.01 * T) for tp in (1, 2) for b in (1, 4) for T in (100, 4000)]
    pred = pat.Predictor(grid)
    table = [(2, r["batch"], r["length"], r["latency_us"]) for r in rows if r["latency_us"] > 0]
    out = pred.pat_switch_decide(1, [1, 2], [(2, 1024.0), (2, 1024.0)], 600, 100, [512] * 4, (2, 256, 2),
                                 {(1, 2): 0.0}, 1.0, 2, prefill=table)     # 1 byte/s network: migration is out
    t_switch = dict((tp, sw) for tp, _, sw, _ in out[4])[2]
    assert t_switch == pytest.approx(lat[(4, 512)], rel=1e-12)


def test_prefill_is_bitwise_repeatable_and_stable_across_pass_widths():
    """The same prompts rebuilt twice give byte-identical K/V (fixed-order reductions everywhere).  A
    different pass width changes which rows share a launch and with that the projection kernel's shape
    (the order of its fp32 partial sums), never which values a row sees: layer 0 agrees to the last
    bf16 bit in all but a handful of elements."""
    pat = _pat()
    shard = pi.CONFIGS["tiny_tp1"]["shard"]
    lens = [130, 37, 64]
    req = pi.rollout_requests(shard, 3, (1, 2), steps=2)
    req["kv_len"] = np.asarray(lens, np.int32)
    toks = np.concatenate([pi.prompt_tokens(shard, i, lens[i]) for i in range(3)])
    outs = []
    for width in (256, 256, 48):
        dec = make_decoder(shard, width, 200, sum(lens) + 64 * 3 + 64, 16)
        dec.pat_decode_admit(req["seq_id"], req["token"], req["kv_len"], req["target"])
        dec.pat_prefill([0, 1, 2], toks)
        outs.append([_kv_bits(dec, j, shard.n_layers, lens[j]) for j in range(3)])
        dec.close()
    for j in range(3):
        for l in range(shard.n_layers):
            for t in range(2):
                assert np.array_equal(outs[0][j][l][t], outs[1][j][l][t])
        for t in range(2):
            same, close = bf16_close(outs[0][j][0][t], outs[2][j][0][t])
            assert close and same > 0.999


# the block attention kernel: every head grouping and head dimension, blocks of 64 / G positions and 64-key tiles cut by
# the sequence ends, pages shorter and longer than a tile
@pytest.mark.parametrize("hq,hkv,d,page,lens,width", [(2, 2, 128, 16, (65, 1, 130), 256), (4, 2, 128, 128, (63, 64, 129), 96),
                                                      (8, 2, 64, 32, (15, 200, 17), 232), (8, 1, 128, 64, (8, 9, 191), 64)])
def test_block_attention_edges(hq, hkv, d, page, lens, width):
    shard = pi.ShardShape(pi.ModelShape(2, 256, hq, hkv, d, 256, 256), 1, 0)
    _prefill_parity(shard, list(lens), list(range(len(lens))), max_batch=width, page_tokens=page, chunked=False)


# few rows over a long context: their keys are cut into chunks and merged; the last pass holds the end of the long sequence
# (several chunks per row) and whole short ones, whose rows take no part in the later chunks
@pytest.mark.parametrize("hq,hkv,d,page,lens,width", [(8, 1, 64, 64, (1300,), 256), (8, 1, 128, 128, (1300, 9, 70), 256),
                                                      (2, 2, 128, 64, (1290, 65), 256), (4, 2, 64, 16, (1400, 1, 130), 256),
                                                      (8, 2, 128, 32, (1100, 33), 128), (2, 2, 64, 64, (900, 20), 128)])
def test_block_attention_over_chunks(hq, hkv, d, page, lens, width):
    shard = pi.ShardShape(pi.ModelShape(2, 256, hq, hkv, d, 256, 256), 1, 0)
    _prefill_parity(shard, list(lens), list(range(len(lens))), max_batch=width, page_tokens=page, steps=1, chunked=True)


# chunks that are no power of two: a wide pass from position 0, and one that begins inside a chunk of its sequence
@pytest.mark.parametrize("hq,hkv,d,page,length,width,chunk", [(8, 4, 128, 16, 700, 700, 192), (16, 16, 64, 128, 900, 512, 192)])
def test_block_attention_over_odd_chunks(hq, hkv, d, page, length, width, chunk):
    shard = pi.ShardShape(pi.ModelShape(2, 256, hq, hkv, d, 256, 256), 1, 0)
    _prefill_parity(shard, [length], [0], max_batch=width, page_tokens=page, steps=1, chunked=True, chunk=chunk)
