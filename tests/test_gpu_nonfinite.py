"""Cached values at and beyond the range of fp32 arithmetic: scores that overflow, positions whose K/V are not numbers."""
import numpy as np
import pytest
import torch

import pat_inputs as pi
from gpu_util import DEV, bf16_close, check_logits
from oracle import Oracle, OracleDecoder, bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,lens,first,n_bad", [
    (8, 1, 128, (100, 33, 200), 0, 32),          # all scores of a wave's first tile of 32 keys
    (4, 1, 64, (100, 300), 0, 32),
    (8, 1, 128, (2600,), 0, 1024),               # ... of the first chunks of a sequence of several
    (8, 2, 64, (2600, 40), 1024, 512),
    (4, 4, 64, (500, 90), 0, 80),                # no grouping
])
def test_keys_whose_scores_overflow_have_no_weight(hq, hkv, d, lens, first, n_bad):
    """Keys `first` .. of every sequence score below -3e38 on every head (query features that rotate slowly are positive,
    those keys' are -3e38): -infinity in fp32, weight zero in the oracle."""
    import paper_2605_23945_amd as pat
    H = 256
    shard = pi.shard_of(pi.ModelShape(1, H, hq, hkv, d, 256, 512), 1, 0)
    tok, n = 7, len(lens)
    slow = slice(d // 2 - d // 16, d // 2)
    w = pi.layer_weights(shard, 0, device=DEV)
    final = pi.final_weights(shard, device=DEV)
    embed = pi.embedding_table(shard, device=DEV)
    toward = torch.sign(embed[tok].float() * w["g1"].float()) * 0.05
    q = torch.zeros(hq, d, H, device=DEV)
    q[:, slow] = toward
    w["wqkv"][: hq * d] = q.view(hq * d, H).to(torch.bfloat16)
    total = int(sum(lens))
    dec = pat.Decoder(pat.make_cfg(shard, n, max(lens) + 4, total + 64 * n, 64), DEV)
    dec.pat_load_layer(0, w)
    dec.pat_load_final(dict(final, embed=embed))
    ids = np.arange(n, dtype=np.int32)
    dec.pat_decode_admit(ids, np.full(n, tok, np.int32), np.array(lens, np.int32), np.full(n, 4, np.int32))
    m = shard.model
    odec = OracleDecoder(Oracle("f64"), (1, H, hq, hkv, d, shard.ffn, m.rms_eps, m.rope_base), lambda l: {k: bits(v.cpu()) for k, v in w.items()},
                         {k: bits(v.cpu()) for k, v in final.items()}, lambda t: bits(embed[t].cpu()))
    for i, L in enumerate(lens):
        k, v = (t.to(DEV).clone() for t in pi.kv_prefix(shard, i, 0, L))
        k[first:first + n_bad, :, slow] = -3.0e38
        dec.pat_kv_write(i, 0, k, v)
        odec.admit(i, tok, L, 4, [bits(k.cpu())], [bits(v.cpu())], 2)
    ref, ref_next, _ = odec.step()
    logits = torch.empty(n, shard.vocab, device=DEV)
    nxt = torch.empty(n, dtype=torch.int32, device=DEV)
    dec.pat_decode_step(True, nxt, logits)
    check_logits(logits.cpu().numpy(), ref)
    assert np.array_equal(nxt.cpu().numpy(), ref_next)
    dec.close()


@pytest.mark.parametrize("hq,hkv,d,length,at,width", [(2, 2, 128, 70, 20, 128), (8, 1, 64, 40, 6, 64), (4, 2, 64, 150, 140, 256),
                                                      (8, 1, 64, 1300, 1293, 256)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_a_position_that_is_not_a_number_leaves_the_earlier_ones_alone(hq, hkv, d, length, at, width, value):
    """Prefill is causal: the states of the positions before `at` do not depend on its token, whose embedding is `value`."""
    import paper_2605_23945_amd as pat
    shard = pi.shard_of(pi.ModelShape(2, 256, hq, hkv, d, 256, 256), 1, 0)
    dec = pat.Decoder(pat.make_cfg(shard, width, length + 4, length + 128, 64), DEV)
    for l in range(2):
        dec.pat_load_layer(l, pi.layer_weights(shard, l, device=DEV))
    embed = pi.embedding_table(shard, device=DEV).clone()
    embed[255] = value
    dec.pat_load_final(dict(pi.final_weights(shard, device=DEV), embed=embed))
    tokens = pi.prompt_tokens(shard, 0, length) % 255
    out = []
    for bad in (False, True):
        t = np.array(tokens, np.int32)
        if bad:
            t[at] = 255
        dec.pat_decode_reset()
        dec.pat_decode_admit([0], [1], [length], [4])
        dec.pat_prefill([0], t)
        out.append([[bits(a.cpu()) for a in dec.pat_kv_read(0, l, length)] for l in range(2)])
    for l in range(2):
        for kv in range(2):
            good, got = out[0][l][kv], out[1][l][kv]
            assert np.all((got[at:].view(np.uint16) & 0x7F80) == 0x7F80) or l == 0     # from `at` on nothing is a number
            # two orders of fp32 sums: the elements near a rounding boundary differ by a bf16 step
            same, close = bf16_close(got[:at], good[:at])
            assert close and same > 0.97, (l, kv, same)
    dec.close()
