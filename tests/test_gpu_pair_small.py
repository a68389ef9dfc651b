"""The multi-hop forward's single launch for the last two hops on small slabs, at its edges: whole and ragged tiles, one and two tiles per
wave, different tile counts for the two hops, grouped heads, narrow rows, every mask, the encoding, and the tensor between the two
hops that a backward needs.  Checked against the oracle and against the hops called one by one."""
import numpy as np
import pytest
import torch

import paper_2410_20926_amd as ta
from gpu_util import TOL, multihop_backward, multihop_forward, to_host
from oracle import tensattn_oracle as orc
from paper_2410_20926_amd.workloads import make_inputs
from grad_bounds import check_backward

pytestmark = pytest.mark.gpu

CASES = [
    # dims, B, Hq, Hkv, D, causal, window, valid_lens, rope base, axes with a table per fibre
    ((5, 10, 9), 1, 3, 3, 128, True, (0, 4, 3), None, None, (2,)),         # 3 and 4 tiles
    ((10, 9), 1, 4, 1, 64, True, None, None, 10000.0, ()),                 # two axes: the value input is per key/value head
    ((12, 8), 2, 4, 2, 128, False, None, (96, 41), None, (0,)),
    ((2, 8, 12), 1, 4, 2, 40, True, None, None, 200.0, ()),                # narrow rows
    ((3, 11, 8), 1, 2, 2, 128, False, (0, 9, 0), None, 10000.0, (1, 2)),   # the encoding at full width, a table per column
    ((4, 16, 8), 2, 8, 2, 64, False, None, (500, 77), None, (1,)),         # whole tiles; one element nearly all padding
    ((16, 16, 16), 2, 8, 2, 128, True, None, (4096, 1500), None, ()),      # 256 slabs: two tiles per wave
    ((18, 15, 16), 2, 8, 8, 40, False, None, None, 10000.0, ()),
    ((32, 20, 8), 1, 8, 2, 128, True, None, (5000,), 10000.0, ()),         # 8 column tiles, 5 row tiles
    ((32, 7, 20), 1, 8, 4, 64, False, None, None, None, (2,)),             # 5 column tiles, 7 row tiles
]


@pytest.mark.parametrize("dims,B,Hq,Hkv,D,causal,window,lens,rope,axes", CASES)
def test_small_slabs_match_oracle_and_single_hops(dims, B, Hq, Hkv, D, causal, window, lens, rope, axes):
    N, m = int(np.prod(dims)), len(dims)
    rng = np.random.default_rng(N + D)
    q, k, v, d_o = make_inputs(B, N, Hq, Hkv, D, seed=8900 + N + D, dtype="bf16", with_grad=True)
    masks = [(rng.random((N // n, n, n)) < 0.7) | np.eye(n, dtype=bool) if i in axes else None for i, n in enumerate(dims)]
    kw = dict(window=window, rope_base=rope)
    pkw = dict(kw, axis_masks=[None if x is None else torch.from_numpy(ta.pack_axis_mask(x)).cuda() for x in masks])
    if lens is not None:
        pkw["valid_lens"] = torch.tensor(lens, dtype=torch.int64, device="cuda")
    okw = dict(kw, valid_len=list(lens) if lens else None, axis_masks=masks)
    got, plan, _ = multihop_forward(q, k, v, dims, "bf16", causal, **pkw)
    saved, plan, dev = multihop_forward(q, k, v, dims, "bf16", causal, save=True, **pkw)
    assert plan.small_pair_position() == m - 2
    ref = orc.tensorized_attention_forward(q, k, v, dims, causal, **okw)
    err = np.abs(got - ref).max()
    assert np.isfinite(got).all() and err <= TOL["bf16"], f"{err:.3e}"
    assert np.array_equal(got, saved)
    # hop by hop: the same roundings in another order of sums
    cur, kind = dev["v"], ta.TA_VIN_KV
    for axis in range(m):
        out = torch.empty_like(dev["o"])
        ta.ta_axis_attn_forward(plan, axis, dev["q"], dev["k"], cur, kind, out)
        if axis == m - 2:                                  # the tensor between the two hops, as kept for the backward
            size = plan.workspace_bytes(True) // (m - 1)
            kept = dev["ws"][axis * size:axis * size + out.numel() * 2].view(torch.bfloat16).view(out.shape)
            assert np.abs(to_host(kept) - to_host(out)).max() <= 1e-2
        cur, kind = out, ta.TA_VIN_O
    torch.cuda.synchronize()
    assert np.abs(to_host(cur) - got).max() <= 1e-2
    grads = multihop_backward(plan, dev, d_o, "bf16")
    check_backward(grads, q, k, v, d_o, dims, causal, "bf16", **okw)
