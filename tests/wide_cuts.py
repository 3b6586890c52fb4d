"""Shapes that reach every kernel of the full-batch projections (33 rows and more), each with the cut it is meant for: (row tiles
of a workgroup, batch tiles of a wave, K slices).  Every slice has 18 k-steps or more, so the weights' ring turns at least once
(its depth is 8 .. 14).  test_wide_projection_cuts.py holds them against the cost model, the GPU tests run them."""
import ctypes

# one projection through the operator entry point: n, k, rows -> cut.  n / 2 is a multiple of 32: all three epilogues run
OPERATORS = {
    (64, 4640, 33): (4, 1, 8), (4288, 640, 65): (4, 1, 1), (1600, 3520, 200): (4, 2, 5),
    (2304, 1280, 200): (8, 1, 2), (6848, 640, 65): (8, 1, 1), (8256, 1728, 65): (8, 2, 3), (24640, 640, 65): (8, 2, 1),
    (3648, 2528, 129): (12, 1, 4), (16448, 640, 65): (12, 1, 1), (5504, 4448, 129): (12, 2, 4), (32832, 640, 65): (12, 2, 1),
    (16448, 3424, 65): (16, 2, 3), (32704, 640, 129): (16, 2, 1),
}

# one layer of a model, a decode step of `rows` sequences: hidden, query heads, KV heads, features, ffn, rows -> cuts by projection
MODELS = {
    (640, 1, 1, 128, 4384, 200): dict(gate_up=(12, 1, 1), down=(4, 1, 6)),
    (640, 4, 1, 64, 6688, 300): dict(gate_up=(12, 2, 1), down=(4, 1, 5)),
    (640, 4, 1, 64, 6624, 500): dict(gate_up=(16, 2, 1), down=(8, 1, 6)),
    (640, 80, 10, 64, 480, 60): dict(o=(4, 1, 8)),
    (640, 1, 1, 128, 2048, 129): dict(gate_up=(8, 1, 1)),
    (640, 2, 2, 64, 4928, 300): dict(gate_up=(8, 2, 1), down=(4, 1, 5)),
    (2560, 2, 2, 128, 672, 500): dict(gate_up=(4, 2, 3), down=(4, 2, 1)),
    (1152, 2, 2, 64, 1760, 129): dict(gate_up=(8, 1, 2), down=(4, 1, 4)),
    (3072, 2, 2, 64, 1664, 300): dict(gate_up=(8, 2, 3), down=(4, 1, 1)),
    (3072, 4, 4, 64, 1472, 200): dict(gate_up=(12, 1, 4), down=(8, 1, 2)),
    (5120, 2, 2, 64, 2848, 150): dict(gate_up=(12, 2, 4), down=(8, 1, 2)),
    (8192, 8, 2, 64, 1216, 1024): dict(gate_up=(16, 2, 3), down=(16, 2, 1)),
    (640, 16, 16, 64, 960, 129): dict(qkv=(4, 1, 1), gate_up=(4, 1, 2)),
    (640, 16, 4, 128, 448, 150): dict(qkv=(8, 1, 1), o=(4, 1, 6)),
    (1152, 10, 10, 128, 448, 129): dict(qkv=(8, 1, 2), o=(4, 1, 4)),
    (640, 12, 12, 128, 576, 700): dict(qkv=(8, 2, 1), o=(4, 1, 2)),
    (1792, 48, 48, 64, 512, 65): dict(qkv=(8, 2, 3), o=(4, 1, 4)),
    (768, 24, 24, 128, 416, 200): dict(qkv=(12, 1, 1), o=(4, 1, 5)),
    (2048, 24, 12, 128, 608, 129): dict(qkv=(12, 1, 2), o=(8, 1, 5)),
    (704, 24, 24, 128, 896, 500): dict(qkv=(12, 2, 1), o=(8, 1, 4)),
    (8192, 6, 6, 128, 736, 1000): dict(qkv=(12, 2, 2), o=(16, 2, 1)),
    (640, 40, 20, 128, 480, 700): dict(qkv=(16, 2, 1), o=(8, 1, 4)),
    (8192, 24, 6, 64, 544, 1024): dict(qkv=(16, 2, 3), o=(16, 2, 1)),
    (1536, 2, 1, 64, 1728, 150): dict(gate_up=(8, 1, 3), down=(4, 1, 3)),
    (768, 64, 8, 64, 864, 129): dict(o=(4, 1, 7), down=(4, 1, 3)),
    (1152, 2, 1, 128, 1376, 300): dict(gate_up=(8, 1, 1), down=(4, 1, 2)),
    (3072, 6, 6, 64, 896, 700): dict(down=(12, 1, 1), gate_up=(8, 1, 1)),
    (6400, 6, 3, 128, 320, 700): dict(o=(12, 2, 1)),
    (4096, 2, 2, 64, 832, 1024): dict(down=(8, 2, 1)),
    (704, 12, 3, 64, 320, 1024): dict(o=(8, 1, 1)),
}
VOCAB = 512


def cut_of(lib, n, k, rows, scratch=None, norm=False):
    c = (ctypes.c_int32 * 5)()
    if scratch is None:
        scratch = lib.pat_op_gemm_scratch_bytes(n, k, rows)
    assert lib.pat_op_gemm_cut(n, k, rows, scratch, int(norm), c) == 0
    return tuple(c)[:3]


def matrices(model):
    h, hq, hkv, d, f, _ = model
    return dict(qkv=((hq + 2 * hkv) * d, h, False), o=(h, hq * d, True), gate_up=(2 * f, h, False), down=(h, f, True), head=(VOCAB, h, False))


def cuts_of(lib, model):
    """As a decoder of that many slots cuts them: the scratch of the largest projection serves all."""
    mats, rows = matrices(model), model[5]
    scratch = max(lib.pat_op_gemm_scratch_bytes(n, k, min(rows, 256)) for n, k, _ in mats.values())
    return {p: cut_of(lib, n, k, rows, scratch, norm) for p, (n, k, norm) in mats.items()}
