"""GPU parity of the resident backward (axes of two to four tiles) at its edges: one row past a tile, whole tiles, three and four
tiles, heads on their own, sharing K, sharing K and the value input, narrow and 64-wide rows, every mask, the encoding, and more fibres
than workgroups (a workgroup then walks several, with the next one's rows on their way)."""
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
    ((33, 65), 1, 2, 2, 128, True, None, None, None),
    ((97, 2), 2, 6, 2, 128, False, None, (150, 31), None),      # groups of three; three tiles and a row; one element nearly all padding
    ((2, 128), 1, 4, 1, 128, True, (0, 20), None, None),        # a band: hidden blocks on both sides
    ((127, 3), 1, 4, 2, 64, False, None, None, 10000.0),
    ((96, 2), 1, 4, 4, 64, True, None, None, None),
    ((3, 70), 1, 3, 1, 100, True, None, (200,), None),          # narrow rows, 8 bytes into an aligned unit for every other head
    ((100, 2), 1, 2, 2, 36, False, None, None, 200.0),
    ((40, 300), 2, 4, 2, 40, True, None, None, None),           # 1,200 fibres and groups: more than are resident at once
    ((260, 48), 1, 4, 2, 128, False, None, None, None),
]


@pytest.mark.parametrize("dims,B,Hq,Hkv,D,causal,window,lens,rope", CASES)
def test_resident_backward_matches_oracle(dims, B, Hq, Hkv, D, causal, window, lens, rope):
    N = int(np.prod(dims))
    q, k, v, d_o = make_inputs(B, N, Hq, Hkv, D, seed=8300 + N + D, dtype="bf16", with_grad=True)
    kw = dict(window=window, rope_base=rope)
    pkw = dict(kw)
    if lens is not None:
        pkw["valid_lens"] = torch.tensor(lens, dtype=torch.int64, device="cuda")
    got, plan, dev = multihop_forward(q, k, v, dims, "bf16", causal, save=True, **pkw)
    ref = orc.tensorized_attention_forward(q, k, v, dims, causal, valid_len=list(lens) if lens else None, **kw)
    assert np.abs(got - ref).max() <= TOL["bf16"]
    axis = int(np.argmax([33 <= n <= 128 for n in dims]))
    assert plan.hop_function(axis, ta.TA_VIN_KV if axis == 0 else ta.TA_VIN_O, True) == "mfma_bwd_resident_kernel"
    grads = multihop_backward(plan, dev, d_o, "bf16")
    check_backward(grads, q, k, v, d_o, dims, causal, "bf16", valid_len=list(lens) if lens else None, **kw)
    again = multihop_backward(plan, dev, d_o, "bf16")
    assert all(np.array_equal(a, b) for a, b in zip(grads, again))          # fixed order of every sum
