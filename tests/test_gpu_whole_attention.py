"""Decode attention of whole sequences (one chunk each, no merge) and the merge of many chunks, through the decode step."""
import numpy as np
import pytest
import torch

import pat_inputs as pi
from gpu_util import DEV, check_logits, make_decoder, make_oracle_decoder, oracle_admit
from test_gpu_step import _gpu_step

pytestmark = pytest.mark.gpu


def _requests(shard, lens):
    req = pi.rollout_requests(shard, len(lens), (1, 2), steps=4)
    req["kv_len"] = np.array(lens, np.int32)
    return req


@pytest.mark.parametrize("hq,hkv,d,page,lens,whole", [
    (4, 4, 64, 16, (0, 1, 62, 63, 64, 127, 128, 188), True),          # whole: more pages than a chunk record holds
    (4, 2, 128, 64, (3, 190, 191, 192), None),                        # the last step crosses from whole sequences to chunks
    (32, 32, 64, 16, (380, 382, 20, 301, 255, 256, 64, 65), None),    # an item per compute unit: whole up to 384
    (8, 1, 128, 16, (100, 311, 30), True),                            # grouped queries
    (2, 2, 128, 64, (1500, 40), False),                                # 24 chunks: four waves merge
    (2, 2, 64, 32, (2500, 2047), False),                               # 40 chunks of 64 features
])
def test_whole_sequences_and_wide_merges_vs_oracle(hq, hkv, d, page, lens, whole):
    import paper_2605_23945_amd as pat
    shard = pi.shard_of(pi.ModelShape(1, 256, hq, hkv, d, 512, 512), 1, 0)
    n = len(lens)
    req = _requests(shard, lens)
    dec = make_decoder(shard, n, max(lens) + 8, int(sum(lens)) + 2 * page * n + 64, page)
    pat.admit_synthetic(dec, shard, req, DEV)
    odec = make_oracle_decoder(shard)
    oracle_admit(odec, shard, req, range(n), 4)
    for _ in range(3):
        assert whole is None or (dec.pat_attention_cut()["step"][1] == n) == whole
        ref_logits, ref_next, _ = odec.step()
        logits, nxt, _ = _gpu_step(dec, n, shard.vocab)
        check_logits(logits, ref_logits)
        assert np.array_equal(nxt, ref_next)
    dec.close()


@pytest.mark.parametrize("hq,hkv,d,page,lens,chunk", [
    (2, 2, 128, 64, (12287, 40), 64),          # 192 chunks
    (2, 2, 128, 64, (12288,), 128),
    (4, 2, 128, 16, (26000, 300), 192),
    (2, 2, 64, 128, (24575,), 128),
    (4, 2, 64, 16, (24600, 1000, 5), 256),
])
def test_long_contexts_take_longer_chunks_vs_oracle(hq, hkv, d, page, lens, chunk):
    shard = pi.shard_of(pi.ModelShape(1, 256, hq, hkv, d, 512, 512), 1, 0)
    import paper_2605_23945_amd as pat
    n, req = len(lens), _requests(shard, lens)
    dec = make_decoder(shard, n, max(lens) + 8, int(sum(lens)) + 2 * page * n + 64, page)
    pat.admit_synthetic(dec, shard, req, DEV)
    odec = make_oracle_decoder(shard)
    oracle_admit(odec, shard, req, range(n), 4)
    assert dec.pat_attention_cut()["step"] == (chunk, sum((l + chunk) // chunk for l in lens))
    ref_logits, ref_next, _ = odec.step()
    logits, nxt, _ = _gpu_step(dec, n, shard.vocab)
    check_logits(logits, ref_logits)
    assert np.array_equal(nxt, ref_next)
    dec.close()


@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 128), (4, 2, 64), (8, 1, 128)])
def test_page_length_does_not_change_a_whole_sequence(hq, hkv, d):
    """The page ids come from the chunk's record or from the wave's lanes; the arithmetic is the same, bit by bit."""
    import paper_2605_23945_amd as pat
    shard = pi.shard_of(pi.ModelShape(1, 256, hq, hkv, d, 512, 512), 1, 0)
    lens = (5, 97, 150, 186)
    out = []
    for page in (16, 32, 64, 128):
        req = _requests(shard, lens)
        dec = make_decoder(shard, len(lens), 256, 1024 + 4 * page * len(lens), page)
        pat.admit_synthetic(dec, shard, req, DEV)
        out.append([_gpu_step(dec, len(lens), shard.vocab)[0] for _ in range(2)])
        dec.close()
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("hq,hkv,d", [(8, 1, 128), (4, 1, 64)])
def test_chunks_of_large_scores_merge_as_one(hq, hkv, d):
    """Scores above ten thousand: a sequence of 300 tokens that is one chunk beside a short one and several beside a long one
    gives the same logits.  The two ways share every score and weight; what differs is the rounding of a few sums and of
    factors near 1 (2^-24 each).  Through it one operand element in about a hundred takes another low term (2^-16 of
    itself), in four operands in turn (attention output, both norms, SwiGLU): 3e-6 of the logits' scale, 3.5 times that for
    the largest of 512, and 2^-15 with a margin of three.  A maximum rounded by 2^-24 of itself is off by 5e-4."""
    import paper_2605_23945_amd as pat
    H = 256
    shard = pi.shard_of(pi.ModelShape(1, H, hq, hkv, d, 256, 512), 1, 0)
    tok = 7
    slow = slice(d // 2 - d // 16, d // 2)
    w = pi.layer_weights(shard, 0, device=DEV)
    embed = pi.embedding_table(shard, device=DEV)
    q = w["wqkv"][: hq * d].view(hq, d, H).clone()
    q[:, slow] = (torch.sign(embed[tok].float() * w["g1"].float()) * 4.0).to(torch.bfloat16)
    w["wqkv"][: hq * d] = q.view(hq * d, H)
    out = []
    for other in (100, 3000):
        lens = (300, other)
        dec = pat.Decoder(pat.make_cfg(shard, 2, 3010, 3600, 64), DEV)
        dec.pat_load_layer(0, w)
        dec.pat_load_final(dict(pi.final_weights(shard, device=DEV), embed=embed))
        dec.pat_decode_admit([0, 1], [tok, tok], lens, [4, 4])
        for i, L in enumerate(lens):
            k, v = (t.to(DEV).clone() for t in pi.kv_prefix(shard, i, 0, L))
            k[:, :, slow] = 20.0
            dec.pat_kv_write(i, 0, k, v)
        chunk, chunks = dec.pat_attention_cut()["step"]
        assert chunks == 2 if other == 100 else 301 > 2 * chunk
        logits = torch.empty(2, shard.vocab, device=DEV)
        dec.pat_decode_step(True, torch.empty(2, dtype=torch.int32, device=DEV), logits)
        out.append(logits[0].double().cpu().numpy())
        dec.close()
    err = float(np.max(np.abs(out[0] - out[1])) / out[0].std())
    print("merge against one chunk:", err, flush=True)
    assert err <= 2.0 ** -15


@pytest.mark.parametrize("heads,n,longest,chunk", [
    (16, 40, 1290, 192),           # 300 MB of K and V: chunks of three rounds
    (16, 61, 1420, 384),           # 500 MB: two workgroups per compute unit, chunks past a record's four pages
    (32, 130, 700, 0),             # 16 items per compute unit: whole sequences
])
def test_long_streams_equal_the_same_sequences_in_a_short_batch(heads, n, longest, chunk):
    """Rows of a batch whose K and V are hundreds of megabytes against the same sequences alone, which are cut into chunks of one
    round.  The sums' order differs, and the projections' kernels (more than 32 rows, at most 32): both are within 1e-4 of the
    logits' scale of float64 in their own tests."""
    _rows_of_a_long_batch(heads, heads, 128, n, longest, chunk, 64)


@pytest.mark.parametrize("hq,hkv,d,n,longest,chunk,page", [
    (16, 16, 128, 40, 1290, 192, 128),         # chunks begin inside a page
    (16, 16, 128, 61, 1420, 384, 16),          # 24 pages per chunk, from the wave's lanes
    (32, 32, 128, 130, 700, 0, 16),
    (32, 32, 128, 150, 400, 0, 64),            # whole, four workgroups per compute unit
    (16, 8, 128, 80, 1290, 320, 64),           # two query heads: five pages
    (16, 8, 128, 80, 1290, 320, 128),
    (16, 8, 128, 130, 1000, 0, 16),            # four items per compute unit: whole, 63 pages
    (16, 8, 64, 60, 1290, 384, 32),
    (16, 8, 64, 130, 900, 0, 128),
    (32, 32, 64, 60, 1000, 128, 16),           # 64 features, one query head: a round whatever the bytes
])
def test_cuts_of_long_batches_and_page_lengths(hq, hkv, d, n, longest, chunk, page):
    """As above, over heads, features and page lengths."""
    _rows_of_a_long_batch(hq, hkv, d, n, longest, chunk, page)


def _rows_of_a_long_batch(hq, hkv, d, n, longest, chunk, page):
    import paper_2605_23945_amd as pat
    shard = pi.shard_of(pi.ModelShape(1, 256, hq, hkv, d, 512, 512), 1, 0)
    lens = np.array([longest - (i * longest) // (2 * n) for i in range(n)], np.int32)
    lens[[0, n - 1]] = lens[[n - 1, 0]]
    off = np.concatenate(([0], np.cumsum(lens)))
    g = torch.Generator(device=DEV).manual_seed(n)
    kv = torch.empty(1, 2, hkv, int(off[-1]), d, dtype=torch.bfloat16, device=DEV).normal_(0, 1, generator=g)
    weights, final = pi.layer_weights(shard, 0, device=DEV), pi.final_weights(shard, device=DEV)
    final = dict(final, embed=pi.embedding_table(shard, device=DEV))

    def step(slots):
        m = len(slots)
        ls = lens[slots]
        dec = pat.Decoder(pat.make_cfg(shard, m, longest + 4, int(ls.sum()) + 2 * page * m, page), DEV)
        dec.pat_load_layer(0, weights)
        dec.pat_load_final(final)
        dec.pat_decode_admit(list(range(m)), [int(3 + 7 * s) % 512 for s in slots], ls, [4] * m)
        buf = kv if m == n else torch.cat([kv[:, :, :, off[s]: off[s + 1]] for s in slots], dim=3).contiguous()
        dec.pat_kv_inject(list(range(m)), buf, layer0=0)
        cut = tuple(int(c) for c in dec.pat_attention_cut()["step"])
        logits = torch.empty(m, shard.vocab, device=DEV)
        dec.pat_decode_step(False, torch.empty(m, dtype=torch.int32, device=DEV), logits)
        out = logits.double().cpu().numpy()
        dec.close()
        return cut, out

    cut, out = step(list(range(n)))
    assert cut == ((longest + 1, n) if chunk == 0 else (chunk, int(sum((l + chunk) // chunk for l in lens))))
    rows = [0, n // 2, n - 1]
    short, ref = step(rows)
    assert short[0] == (64 if d == 128 else 128)
    assert np.max(np.abs(out[rows] - ref)) <= 2e-4 * float(ref.std())


@pytest.mark.parametrize("hq,hkv,d,n,length,period,page", [
    (32, 32, 128, 8, 383, 384, 64),            # an item per compute unit: whole sequences of 384
    (32, 16, 128, 16, 383, 384, 128),
    (32, 32, 64, 8, 383, 384, 32),
    (32, 16, 64, 16, 383, 384, 16),
    (16, 16, 128, 80, 1151, 384, 64),          # 700 MB: three chunks of 384
    (32, 32, 128, 130, 1023, 1024, 16),        # 16 items per compute unit: whole sequences of 1024, 64 pages each
])
def test_terms_of_a_long_chunk_are_not_lost_beside_its_large_sums(hq, hkv, d, n, length, period, page):
    """All keys are zero, so every weight is 1.  Of `period` values the first 128 are 2^20, the last 128 -2^20, those between
    1/8: a lane's sum of the first is 2^22 or 2^23, where one 1/8 after another is rounded away and 4 or 8 of them together
    (128 tokens) are exact.  The last token is the appended one, whose value is zero; its lane has one 2^20 less too."""
    import paper_2605_23945_amd as pat
    H, tok, rows = 256, 7, 2048 // d                # token rows that a lane position of the kernel stands for
    shard = pi.shard_of(pi.ModelShape(1, H, hq, hkv, d, 256, 512), 1, 0)
    w = {k: v.clone() for k, v in pi.layer_weights(shard, 0, device=DEV).items()}
    w["wqkv"][hq * d:] = 0
    w["wd"][:] = 0
    final, embed = pi.final_weights(shard, device=DEV), pi.embedding_table(shard, device=DEV)
    t = torch.arange(length, device=DEV) % period
    small = (t >= 128) & (t < period - 128)
    value = torch.where(t < 128, 2.0 ** 20, torch.where(small, 0.125, -2.0 ** 20))
    value[(t == rows - 1) | (t == period - 1)] = 0
    sign = torch.randint(0, 2, (d,), generator=torch.Generator().manual_seed(3)).to(DEV) * 2.0 - 1.0
    kv = torch.zeros(1, 2, hkv, length * n, d, dtype=torch.bfloat16, device=DEV)
    kv[0, 1] = (value[:, None] * sign).to(torch.bfloat16).repeat(n, 1)
    dec = pat.Decoder(pat.make_cfg(shard, n, length + 4, n * (length + 2 * page), page), DEV)
    dec.pat_load_layer(0, w)
    dec.pat_load_final(dict(final, embed=embed))
    dec.pat_decode_admit(list(range(n)), [tok] * n, [length] * n, [4] * n)
    dec.pat_kv_inject(list(range(n)), kv, layer0=0)
    assert dec.pat_attention_cut()["step"] == (period, n * (length + 1) // period)
    logits = torch.empty(n, shard.vocab, device=DEV)
    dec.pat_decode_step(False, torch.empty(n, dtype=torch.int32, device=DEV), logits)
    o = 0.125 * float(small.sum()) / (length + 1) * sign.double().repeat(hq)
    x = embed[tok].double() + w["wo"].double() @ o
    x = x / torch.sqrt((x * x).mean() + shard.model.rms_eps) * final["gf"].double()
    check_logits(logits.cpu().numpy(), (final["wlm"].double() @ x).cpu().numpy()[None].repeat(n, 0))
    dec.close()
