"""The full-batch projection kernel (33 rows and more) at the edges of its tiles, rings, row groups and K slices, through the
C ABI, against float64 products of the same operands."""
import numpy as np
import pytest
import torch

import pat_inputs as pi
from gpu_util import DEV
from test_gpu_step import _sampled_rows_parity
from wide_cuts import MODELS, OPERATORS, VOCAB, cut_of, cuts_of

pytestmark = pytest.mark.gpu

# rows: both sides of every batch-tile count; row tiles: one, a workgroup's 4 / 8 / 12 / 16 and one more or less, several ranges;
# k-steps: fewer than the rings hold, a multiple of their unrolling and one more or less, slices of unequal length
CASES = [(16, 32, 33), (16, 160, 64), (64, 192, 65), (80, 224, 128), (128, 256, 129), (192, 288, 192), (208, 352, 193),
         (400, 416, 256), (64, 512, 34), (80, 544, 255), (784, 608, 63), (144, 1056, 127), (208, 2080, 191), (1200, 832, 80),
         (3088, 544, 40), (3088, 480, 250), (33024, 96, 36), (33024, 64, 200), (32752, 192, 131), (28688, 224, 250), (32000, 96, 256)]


@pytest.mark.parametrize("n,k,b", CASES)
def test_edges_of_tiles_rings_and_slices(n, k, b):
    _all_epilogues(n, k, b)


@pytest.mark.parametrize("n,k,b", OPERATORS)
def test_every_kernel_past_a_turn_of_its_ring(n, k, b):
    import paper_2605_23945_amd as pat
    assert cut_of(pat.load_library(), n, k, b) == OPERATORS[n, k, b]
    _all_epilogues(n, k, b)


@pytest.mark.parametrize("model", MODELS, ids=lambda m: "-".join(map(str, m)))
def test_every_kernel_with_the_step_s_own_epilogues(model):
    """Rotary embedding and append, residual with the next RMSNorm, SwiGLU, in a decode step of one layer; rows at the edges of
    the batch tiles and row groups."""
    import paper_2605_23945_amd as pat
    h, hq, hkv, d, f, rows = model
    got = cuts_of(pat.load_library(), model)
    assert all(got[p] == c for p, c in MODELS[model].items()), got
    shard = pi.shard_of(pi.ModelShape(1, h, hq, hkv, d, f, VOCAB), 1, 0)
    edges = sorted({0, 15, 16, min(63, rows - 2), (rows // 2) & ~15, rows - 1})
    _sampled_rows_parity(shard, rows, (1, 6), edges, page_tokens=16)


def _all_epilogues(n, k, b):
    import paper_2605_23945_amd as pat
    lib = pat.load_library()
    w = pi.normal_bf16(pi.stream_key(0x31DE, n, k), torch.arange(n * k, dtype=torch.int64, device=DEV), 0.05).view(n, k)
    x = torch.randn(b, k, device=DEV, generator=torch.Generator(device=DEV).manual_seed(b))
    hi, lo = pat.pat_op_pack_act(x)
    ref = x.double().cpu().numpy() @ w.double().cpu().numpy().T
    # operands hi + lo are good to 2^-17, sums are fp32: a few units of 2^-17 of the row scale (the same bound as the
    # other projection tests)
    tol = 1e-4 * float(np.sqrt(np.mean(ref * ref)))
    wp = pat.pat_op_pack_weight(w)
    y = torch.full((b, n), 7.0, device=DEV)
    pat.pat_op_gemm(wp, n, k, hi, lo, b, y, mode=0)
    assert np.max(np.abs(y.double().cpu().numpy() - ref)) <= tol
    y2 = torch.full((b, n), 0.25, device=DEV)
    pat.pat_op_gemm(wp, n, k, hi, lo, b, y2, mode=1)
    assert np.max(np.abs(y2.double().cpu().numpy() - 0.25 - ref)) <= tol + 1e-6
    if (n // 2) % 32 == 0:
        wg = pat.pat_op_pack_weight(w[: n // 2], w[n // 2:])
        nb = lib.pat_op_packed_act_bytes(b, n // 2)
        yh = torch.zeros(nb, dtype=torch.uint8, device=DEV)
        yl = torch.zeros_like(yh)
        pat.pat_op_gemm(wg, n, k, hi, lo, b, None, mode=2, y_hi=yh, y_lo=yl)
        g, u = ref[:, : n // 2], ref[:, n // 2:]
        want = g / (1.0 + np.exp(-g)) * u
        assert np.max(np.abs(pat.unpack_act(yh, yl, b, n // 2) - want)) <= 2e-4 * float(np.sqrt(np.mean(want * want))) + 2 * tol * float(np.max(np.abs(ref)))


@pytest.mark.parametrize("n,k,b", [(22016, 4096, 40), (22016, 4096, 256), (32000, 4096, 200), (13824, 5120, 101), (7168, 8192, 60),
                                   (7168, 8192, 256), (4096, 11008, 128)])
def test_long_sums_are_taken_in_blocks(n, k, b):
    """The fp32 sums against float64 sums of the same split operands.  A rounding of the running sum costs about 2.5e-8 of it
    (2^-24 uniform, averaged over a binade); blocks of at most 15 k-steps and a second chain over the blocks stay below
    2.2e-7, one chain of 2 k / 32 additions gives 4e-7 .. 8e-7 at these depths."""
    import paper_2605_23945_amd as pat
    g = torch.Generator(device=DEV).manual_seed(n + k + b)
    w = torch.empty(n, k, dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
    x = torch.randn(b, k, device=DEV, generator=g)
    hi, lo = pat.pat_op_pack_act(x)
    y = torch.empty(b, n, device=DEV)
    pat.pat_op_gemm(pat.pat_op_pack_weight(w), n, k, hi, lo, b, y, mode=0)
    xh = x.bfloat16().float()
    xl = (x - xh).bfloat16().float()
    ref = (xh.double() + xl.double()) @ w.double().t().contiguous()
    err = float((y.double() - ref).norm() / ref.norm())
    print(f"{n} x {k}, {b} rows: {err:.3e}", flush=True)
    assert err <= 2.2e-7
