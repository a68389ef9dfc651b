"""Long-axis forward with sequences that end early: workgroups of nothing but padding, of some padding, and none, in step and in phases, heads that share
K or do not.  Padding is zero in the output, the rest as the oracle has it."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, multihop_forward
from oracle import tensattn_oracle as orc
from paper_2410_20926_amd.workloads import make_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # axis, Hq, Hkv, D, causal, lens, form
    (2311, 2, 2, 128, True, (2311, 256, 1), "four_tiles_in_step"),   # (too few workgroups for eight tiles each)
    (2304, 32, 32, 64, False, (1200, 2049), "eight_tiles_in_phases"),   # one head per workgroup
    (2304, 128, 32, 128, True, (700, 65), "eight_tiles_in_phases"),   # four heads per workgroup
    (4130, 16, 16, 40, True, (4130, 1000), "eight_tiles_in_phases"),   # narrow rows
]


@pytest.mark.parametrize("n,Hq,Hkv,D,causal,lens,form", CASES)
def test_sequences_that_end_early(n, Hq, Hkv, D, causal, lens, form):
    B = len(lens)
    q, k, v = make_inputs(B, n, Hq, Hkv, D, seed=9700 + n + D, dtype="bf16")
    got, plan, _ = multihop_forward(q, k, v, (n,), "bf16", causal, valid_lens=torch.tensor(lens, dtype=torch.int64, device="cuda"))
    assert plan.hop_function(0, 0) == "mfma_fwd_long_kernel" and plan.hop_form(0, 0) == form
    assert np.isfinite(got).all() and all(not got[b, x:].any() for b, x in enumerate(lens))
    h = [0, Hq - 1]                                        # the oracle on the first and the last head
    g = [x // (Hq // Hkv) for x in h]
    ref = orc.tensorized_attention_forward(np.ascontiguousarray(q[:, :, h]), np.ascontiguousarray(k[:, :, g]), np.ascontiguousarray(v[:, :, g]), (n,), causal, valid_len=list(lens))
    assert np.abs(got[:, :, h] - ref).max() <= TOL["bf16"]
