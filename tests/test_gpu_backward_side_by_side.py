"""GPU parity of the one-tile backward where heads have no group and one, two or four of them share a workgroup: one in small calls, compared with
the oracle (whole and narrow rows, packed and ragged tiles, masks, the encoding, a partial last tile); two or four in calls that fill the chip, compared
bit for bit with each head in a call of its own, where it has a workgroup to itself."""
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
    # dims, B, heads, D, causal, window, valid_lens, rope base, axes with a table
    ((7, 32), 1, 1, 128, True, None, None, None, ()),
    ((9, 11), 2, 2, 64, False, None, (99, 40), None, ()),
    ((31, 5), 1, 3, 128, True, (4, 0), None, None, (1,)),
    ((3, 6, 17), 1, 4, 64, True, None, None, 10000.0, ()),
    ((16, 13), 1, 6, 100, False, None, None, None, (0,)),
    ((5, 32), 2, 8, 100, True, None, (160, 33), None, ()),
    ((20, 9), 1, 12, 128, False, None, None, 500.0, ()),
    ((4, 4, 10), 1, 5, 40, True, None, None, None, ()),
    ((32, 2), 1, 16, 20, True, None, None, None, ()),
]


@pytest.mark.parametrize("dims,B,H,D,causal,window,lens,rope,axes", CASES)
def test_ungrouped_heads_match_oracle(dims, B, H, D, causal, window, lens, rope, axes):
    N = int(np.prod(dims))
    rng = np.random.default_rng(N + H)
    q, k, v, d_o = make_inputs(B, N, H, H, D, seed=9100 + N + H, dtype="bf16", with_grad=True)
    masks = [(rng.random((n, n)) < 0.7) | np.eye(n, dtype=bool) if i in axes else None for i, n in enumerate(dims)]
    kw = dict(window=window, rope_base=rope)
    pkw = dict(kw, axis_masks=[None if x is None else torch.from_numpy(ta.pack_axis_mask(x)).cuda() for x in masks])
    if lens is not None:
        pkw["valid_lens"] = torch.tensor(lens, dtype=torch.int64, device="cuda")
    okw = dict(kw, valid_len=list(lens) if lens else None, axis_masks=masks)
    got, plan, dev = multihop_forward(q, k, v, dims, "bf16", causal, save=True, **pkw)
    assert np.abs(got - orc.tensorized_attention_forward(q, k, v, dims, causal, **okw)).max() <= TOL["bf16"]
    assert plan.hop_function(0, ta.TA_VIN_KV, True) == "mfma_bwd_kernel"
    grads = multihop_backward(plan, dev, d_o, "bf16")
    check_backward(grads, q, k, v, d_o, dims, causal, "bf16", **okw)
    again = multihop_backward(plan, dev, d_o, "bf16")
    assert all(np.array_equal(a, b) for a, b in zip(grads, again))


@pytest.mark.parametrize("dims,B,H,D,causal,window,lens,rope,axes", [
    ((31, 16), 2, 60, 128, True, None, None, None, ()),     # 1,860 waves on the second axis: four heads side by side
    ((32, 25), 4, 26, 64, False, None, (800, 431, 32, 1), None, ()),   # two: 26 heads do not divide by four
    ((20, 30), 4, 36, 64, True, (0, 5), None, 500.0, (0,)),
    ((29, 27), 4, 12, 100, True, None, None, None, (1,)),   # narrow rows, 324 and 348 workgroups of one head a sequence, no multiple of eight: two
    ((10, 27), 12, 12, 40, False, (3, 0), None, 500.0, ()), # the same on tiles of three fibres; the other axis, 120, one
    ((27, 30), 2, 40, 100, True, None, None, None, (1,)),   # narrow rows in order: one
    ((17, 31), 3, 45, 20, False, None, None, None, ()),     # 45 heads: one
])
def test_heads_side_by_side_give_the_bits_of_heads_alone(dims, B, H, D, causal, window, lens, rope, axes):
    N = int(np.prod(dims))
    rng = np.random.default_rng(N + H)
    q, k, v, d_o = make_inputs(B, N, H, H, D, seed=9200 + N + H, dtype="bf16", with_grad=True)
    kw = dict(window=window, rope_base=rope, axis_masks=[torch.from_numpy(ta.pack_axis_mask((rng.random((n, n)) < 0.7) | np.eye(n, dtype=bool))).cuda()
                                                         if i in axes else None for i, n in enumerate(dims)])
    if lens is not None:
        kw["valid_lens"] = torch.tensor(lens, dtype=torch.int64, device="cuda")

    def step(h):
        _, plan, dev = multihop_forward(*(np.ascontiguousarray(t[:, :, h]) for t in (q, k, v)), dims, "bf16", causal, save=True, **kw)
        return multihop_backward(plan, dev, np.ascontiguousarray(d_o[:, :, h]), "bf16")
    forms = [ta.ta_plan_create(B, H, H, D, dims, ta.TA_BF16, causal, **kw).hop_form(i, ta.TA_VIN_KV, True) for i in range(len(dims))]
    assert forms == {(100, 12): ["heads_in_pairs"] * 2, (40, 12): ["heads_in_pairs", "rows_cached"]}.get((D, H), ["rows_cached" if D not in (64, 128) else ""] * 2)
    whole = step(slice(None))
    assert all(np.isfinite(x).all() for x in whole)
    for h in (0, 1, 2, 3, H // 2, H - 2, H - 1):
        assert all(np.array_equal(x[:, :, h:h + 1], y) for x, y in zip(whole, step(slice(h, h + 1)))), h


@pytest.mark.parametrize("dims,axis,B,H,Hkv,D,rope", [
    ((32, 150), 0, 4, 16, 16, 100, None),                  # 430 MB in a hop, a quarter of it in a sequence
    ((300, 11), 1, 8, 16, 4, 96, 10000.0),                 # a group, tiles of two fibres, encoded
    ((32, 220), 0, 4, 32, 2, 40, None),                    # two launches per group
])
def test_streamed_narrow_rows_give_the_bits_of_cached_ones(dims, axis, B, H, Hkv, D, rope):
    N, gen = int(np.prod(dims)), torch.Generator(device="cuda").manual_seed(9300 + D)
    q, g, x = (torch.randn((B, N, H, D), generator=gen, device="cuda").bfloat16() for _ in range(3))
    k = torch.randn((B, N, Hkv, D), generator=gen, device="cuda").bfloat16()

    def hop(form, *rows):
        plan = ta.ta_plan_create(rows[0].shape[0], H, Hkv, D, dims, ta.TA_BF16, True, rope_base=rope)
        assert plan.hop_form(axis, ta.TA_VIN_O, True) == form
        grads = [torch.full_like(t, 0.5) for t in (rows[0], rows[1], rows[2])]
        for accumulate in (False, True):
            ta.ta_axis_attn_backward(plan, axis, rows[0], rows[1], rows[2], ta.TA_VIN_O, rows[3], grads[2], grads[0], grads[1], accumulate)
        return grads
    whole = hop("rows_streamed", q, k, x, g)
    for b in (0, B - 1):
        part = hop("rows_cached", *(t[b:b + 1].contiguous() for t in (q, k, x, g)))
        assert all(torch.isfinite(y).all() and torch.equal(y[b:b + 1], z) for y, z in zip(whole, part))
