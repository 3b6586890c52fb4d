"""The projections of at most 8 rows, where a row's high and low terms share one matrix operand, through the C ABI."""
import numpy as np
import pytest
import torch

import pat_inputs as pi
from gpu_util import DEV

pytestmark = pytest.mark.gpu

# rows: one, both sides of the half tile (9 rows take the kernel of 9..16); row tiles: one, one per workgroup, more than
# a workgroup's eight; k-steps: fewer than the waves, one pass, passes with every kind of remainder
CASES = [(16, 32, 1), (48, 96, 8), (80, 512, 7), (4096, 4096, 8), (208, 4608, 3), (272, 11008, 2), (144, 6944, 5), (33040, 160, 8)]


@pytest.mark.parametrize("n,k,b", CASES)
def test_up_to_eight_rows_equal_the_same_rows_of_a_larger_batch(n, k, b):
    """Same operands, same order of sums: the first rows of a batch of 9 to 16 (another kernel) agree bit by bit, and both
    agree with float64 (operands hi + lo are good to 2^-17, sums are fp32: the bound of the other projection tests)."""
    import paper_2605_23945_amd as pat
    w = pi.normal_bf16(pi.stream_key(0x5A11, n, k), torch.arange(n * k, dtype=torch.int64, device=DEV), 0.05).view(n, k)
    x = torch.randn(9 + b % 8, k, device=DEV, generator=torch.Generator(device=DEV).manual_seed(b))
    wp = pat.pat_op_pack_weight(w)

    def project(rows, mode, fill):
        hi, lo = pat.pat_op_pack_act(rows.contiguous())
        y = torch.full((len(rows), n), fill, device=DEV)
        pat.pat_op_gemm(wp, n, k, hi, lo, len(rows), y, mode=mode)
        return y

    y = project(x[:b], 0, 7.0)
    assert torch.equal(y, project(x, 0, 7.0)[:b])
    assert torch.equal(project(x[:b], 1, 0.25), project(x, 1, 0.25)[:b])
    ref = x[:b].double().cpu().numpy() @ w.double().cpu().numpy().T
    assert np.max(np.abs(y.double().cpu().numpy() - ref)) <= 1e-4 * float(np.sqrt(np.mean(ref * ref)))
