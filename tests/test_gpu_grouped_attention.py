"""Decode attention of grouped queries (4 or 8 query heads per KV head) at the edges of its tiles: 32 keys per wave and
turn, four waves, 16-key halves that may lie in different pages, chunks whose last wave has no tile."""
import numpy as np
import pytest

import pat_inputs as pi
from gpu_util import DEV, check_logits, make_decoder, make_oracle_decoder, oracle_admit
from test_gpu_step import _gpu_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,page,lens", [
    (8, 1, 128, 64, (0, 1, 15, 16, 31, 32, 33, 63, 64, 95, 96, 127, 128)),      # every wave's first and last tile
    (8, 1, 128, 16, (14, 47, 64, 80, 600)),                                     # halves of a tile in two pages
    (4, 1, 64, 128, (30, 127, 128, 129, 700)),
    (16, 2, 64, 32, (1, 62, 200, 333)),                                         # 8 heads on each of two KV heads
    (8, 2, 128, 64, (2, 255, 1021)),
])
def test_decode_attention_of_grouped_queries(hq, hkv, d, page, lens):
    import paper_2605_23945_amd as pat
    shard = pi.shard_of(pi.ModelShape(1, 256, hq, hkv, d, 512, 512), 1, 0)
    n = len(lens)
    req = pi.rollout_requests(shard, n, (1, 2), steps=4)
    req["kv_len"] = np.array(lens, np.int32)
    dec = make_decoder(shard, n, max(lens) + 8, int(sum(lens)) + 2 * page * n + 64, page)
    pat.admit_synthetic(dec, shard, req, DEV)
    odec = make_oracle_decoder(shard)
    oracle_admit(odec, shard, req, range(n), 4)
    for _ in range(3):
        ref_logits, ref_next, _ = odec.step()
        logits, nxt, _ = _gpu_step(dec, n, shard.vocab)
        check_logits(logits, ref_logits)
        assert np.array_equal(nxt, ref_next)
    dec.close()


@pytest.mark.parametrize("hq,hkv,d,n,longest,chunk", [(8, 1, 128, 24, 1500, 192), (8, 1, 128, 36, 2000, 320), (8, 1, 128, 40, 2600, 448),
                                                      (4, 1, 128, 3, 700, 64)])
def test_chunks_that_start_inside_a_page(hq, hkv, d, n, longest, chunk):
    """Pages of 128 tokens and chunks that are no multiple of them: a chunk's first key lies in the middle of a page, and its
    pages are one more than its length suggests."""
    import paper_2605_23945_amd as pat
    shard = pi.shard_of(pi.ModelShape(1, 256, hq, hkv, d, 512, 512), 1, 0)
    lens = np.array([longest - 7 * i for i in range(n)], np.int32)
    req = pi.rollout_requests(shard, n, (1, 2), steps=4)
    req["kv_len"] = lens
    dec = make_decoder(shard, n, longest + 8, int(lens.sum()) + 256 * n, 128)
    pat.admit_synthetic(dec, shard, req, DEV)
    rows = sorted({0, 1, n // 2, n - 1})
    odec = make_oracle_decoder(shard)
    oracle_admit(odec, shard, req, rows, 4)
    for _ in range(2):
        assert dec.pat_attention_cut()["step"][0] == chunk
        ref_logits, ref_next, _ = odec.step()
        logits, nxt, _ = _gpu_step(dec, n, shard.vocab)
        check_logits(logits[rows], ref_logits)
        assert np.array_equal(nxt[rows], ref_next)
    dec.close()
