"""GPU parity of the long-axis backward at its edges: five tiles (one row in the last), whole blocks, a block and a row, more than
eight tiles (several rounds), groups that share K and the value input, more than eight heads per group (several launches), narrow and 64-wide
rows, every mask, the encoding.  And of the blocked kernel, which stays for axes of five and six tiles whose heads come in groups of four or more
and that fill the chip, or of eight or more on five tiles: every tile width, every mask, the encoding, more than eight heads per group."""
import numpy as np
import pytest
import torch

import paper_2410_20926_amd as ta
from gpu_util import TOL, multihop_backward, multihop_forward
from oracle import tensattn_oracle as orc
from paper_2410_20926_amd.workloads import make_inputs
from grad_bounds import check_backward

pytestmark = pytest.mark.gpu

CASES = [
    # dims, B, Hq, Hkv, D, causal, window, valid_lens, rope base
    ((129, 2), 1, 2, 2, 128, True, None, None, None),
    ((2, 192), 1, 4, 2, 128, False, None, None, None),
    ((257,), 2, 3, 1, 64, True, None, (257, 40), None),
    ((300, 2), 1, 2, 1, 100, False, (50, 0), None, 10000.0),
    ((2, 320), 1, 2, 2, 36, True, None, (500,), None),
    ((513,), 1, 1, 1, 128, True, None, None, 10000.0),
    ((170, 3), 1, 18, 2, 64, True, None, None, None),          # nine heads per group: two launches
    ((200,), 1, 8, 2, 128, False, (70,), None, None),
]
BLOCKED = [
    # ... and whether the long axis has a table per fibre
    ((161, 70), 1, 16, 4, 64, True, None, None, None, False),
    ((130, 64), 1, 16, 4, 128, True, None, None, 10000.0, False),
    ((129, 64), 2, 8, 2, 100, False, None, (129 * 64, 3000), None, True),      # narrow rows in 128-wide tiles
    ((192, 64), 1, 16, 4, 40, True, (50, 0), None, 200.0, False),              # six whole tiles; narrow rows in 64-wide ones
    ((130, 128), 1, 18, 2, 40, False, None, (9000,), None, False),             # nine heads per group: two launches
    ((160, 2), 1, 8, 1, 128, True, None, None, None, False),                   # eight heads per group: on any number of fibres
    ((66, 150), 1, 16, 4, 128, False, (0, 33), None, None, True),              # per-head value input
]


@pytest.mark.parametrize("dims,B,Hq,Hkv,D,causal,window,lens,rope,table,function",
                         [(*c, False, "mfma_bwd_long_kernel") for c in CASES] + [(*c, "mfma_bwd_stream_kernel") for c in BLOCKED])
def test_long_backward_matches_oracle(dims, B, Hq, Hkv, D, causal, window, lens, rope, table, function):
    N, axis = int(np.prod(dims)), int(np.argmax(dims))
    n = dims[axis]
    q, k, v, d_o = make_inputs(B, N, Hq, Hkv, D, seed=8700 + N + D, dtype="bf16", with_grad=True)
    kw = dict(window=window, rope_base=rope)
    pkw = dict(kw)
    if table:
        seen = (np.random.default_rng(n).random((N // n, n, n)) < 0.7) | np.eye(n, dtype=bool)
        kw["axis_masks"] = [seen if i == axis else None for i in range(len(dims))]
        pkw["axis_masks"] = [torch.from_numpy(ta.pack_axis_mask(seen)).cuda() if i == axis else None for i in range(len(dims))]
    if lens is not None:
        pkw["valid_lens"] = torch.tensor(lens, dtype=torch.int64, device="cuda")
    got, plan, dev = multihop_forward(q, k, v, dims, "bf16", causal, save=True, **pkw)
    ref = orc.tensorized_attention_forward(q, k, v, dims, causal, valid_len=list(lens) if lens else None, **kw)
    assert np.abs(got - ref).max() <= TOL["bf16"]
    assert plan.hop_function(axis, ta.TA_VIN_KV if axis == 0 else ta.TA_VIN_O, True) == function
    grads = multihop_backward(plan, dev, d_o, "bf16")
    check_backward(grads, q, k, v, d_o, dims, causal, "bf16", valid_len=list(lens) if lens else None, **kw)
    again = multihop_backward(plan, dev, d_o, "bf16")
    assert all(np.array_equal(a, b) for a, b in zip(grads, again))          # fixed order of every sum
