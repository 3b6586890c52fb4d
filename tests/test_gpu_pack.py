"""The streaming layout of a weight matrix, byte by byte: k-steps that are no multiple of a wave's four, rows that are no
multiple of a tile, gate/up pairs."""
import numpy as np
import pytest
import torch

from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,pair", [(16, 32, False), (40, 96, False), (100, 160, False), (33, 224, False), (2064, 4096, False),
                                      (8, 32, True), (20, 288, True), (1376, 544, True)])
def test_packed_bytes(n, k, pair):
    import paper_2605_23945_amd as pat
    g = torch.Generator().manual_seed(n + k)
    w = torch.randn((2, n, k) if pair else (n, k), generator=g).to(torch.bfloat16)
    got = pat.pat_op_pack_weight(*(w.to(DEV) if pair else [w.to(DEV)])).cpu()
    rows = w.transpose(0, 1).reshape(2 * n, k) if pair else w                  # rows of a pair alternate
    src = rows.contiguous().view(torch.int16).numpy()
    full = np.zeros((-(-len(src) // 16) * 16, k), np.int16)
    full[: len(src)] = src
    # vector (tile, k-step, lane): row 16 tile + lane % 16, eight features from 32 k-step + 8 (lane / 16)
    want = full.reshape(-1, 16, k // 32, 4, 8).transpose(0, 2, 3, 1, 4)
    assert np.array_equal(got.view(torch.int16).numpy().reshape(-1)[: want.size], want.reshape(-1))
