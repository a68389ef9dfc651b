"""fp32 backward of axes of two tiles, where two waves share a tile's key side: an odd and an even number of heads per group, a single head (every second query
tile instead), one row in the second tile, masks that leave a wave without a query tile, and the encoding."""
import numpy as np
import pytest
import torch

import paper_2410_20926_amd as ta
from gpu_util import multihop_backward, multihop_forward
from grad_bounds import check_backward
from paper_2410_20926_amd.workloads import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,H,Hkv,D,causal,window,lens,rope", [
    ((33, 3), 3, 1, 64, True, None, None, None),
    ((2, 64), 4, 1, 128, False, None, (100, 20), None),
    ((40, 5), 2, 2, 100, True, None, None, 10000.0),       # heads on their own
    ((5, 50), 4, 2, 20, False, (0, 10), None, None),       # a band
    ((64, 2), 1, 1, 40, True, (4, 0), None, 300.0),
    ((45, 34), 6, 2, 36, True, None, (700, 1530), None),
])
def test_two_tiles_match_oracle(dims, H, Hkv, D, causal, window, lens, rope):
    N, B = int(np.prod(dims)), 2
    q, k, v, d_o = make_inputs(B, N, H, Hkv, D, seed=9900 + N + D, dtype="f32", with_grad=True)
    kw = dict(window=window, rope_base=rope)
    pkw = dict(kw, valid_lens=torch.tensor(lens, dtype=torch.int64, device="cuda") if lens else None)
    _, plan, dev = multihop_forward(q, k, v, dims, "f32", causal, save=True, **pkw)
    grads = multihop_backward(plan, dev, d_o, "f32")
    check_backward(grads, q, k, v, d_o, dims, causal, "f32", valid_len=list(lens) if lens else None, **kw)
    again = multihop_backward(plan, dev, d_o, "f32")
    assert all(np.array_equal(a, b) for a, b in zip(grads, again))          # fixed order of every sum
