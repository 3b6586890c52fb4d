"""The cost model of the full-batch projections picks the cuts that the GPU tests mean to run, and these are all there are."""
import ctypes

import pytest

import paper_2605_23945_amd as pat
from wide_cuts import MODELS, OPERATORS, cut_of, cuts_of, matrices

SHAPES = [(4, 1), (4, 2), (8, 1), (8, 2), (12, 1), (12, 2), (16, 2)]       # row tiles x batch tiles


def test_operator_shapes_are_cut_as_listed_and_cover_every_kernel():
    lib = pat.load_library()
    for (n, k, rows), want in OPERATORS.items():
        assert cut_of(lib, n, k, rows) == want, (n, k, rows)
        assert (n // 2) % 32 == 0 and k // 32 // want[2] >= 18
    for s in SHAPES:
        slices = {c[2] for c in OPERATORS.values() if c[:2] == s}
        assert max(slices) > 1 and (1 in slices or s == (4, 2)), s


def test_models_are_cut_as_listed_and_cover_every_kernel():
    lib = pat.load_library()
    seen = {}
    for m, want in MODELS.items():
        got, mats = cuts_of(lib, m), matrices(m)
        for p, c in want.items():
            assert got[p] == c, (m, p, got[p])
            if mats[p][1] // 32 // c[2] >= 18:
                seen.setdefault("residual" if p in ("o", "down") else p, set()).add(c)
    for p in ("qkv", "gate_up"):
        whole, sliced = {c[:2] for c in seen[p] if c[2] == 1}, {c[:2] for c in seen[p] if c[2] > 1}
        assert whole >= {s for s in SHAPES if s[0] != 4}, (p, whole)       # four row tiles always write partial sums there
        assert sliced >= {s for s in SHAPES if s[0] != 4}, (p, sliced)
    assert {c[:2] for c in seen["residual"] if c[2] == 1} == set(SHAPES)
    # the reduction with the RMSNorm: one instance per number of slices, one slice of four row tiles among them
    assert {c[2] for c in seen["residual"] if c[2] > 1 or c[0] == 4} == set(range(1, 9))


@pytest.mark.parametrize("args", [(0, 64, 40, 0, 0), (64, 33, 40, 0, 0), (64, 64, 32, 0, 0), (64, 64, 1025, 0, 0), (64, 64, 40, -1, 0)])
def test_cut_query_rejects_bad_arguments(args):
    assert pat.load_library().pat_op_gemm_cut(*args, (ctypes.c_int32 * 5)()) == pat.binding.PAT_EINVAL
