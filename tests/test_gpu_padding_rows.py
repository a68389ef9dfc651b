"""A forward hop along an axis of up to 64 positions does not read padding: tokens at or past a sequence's length hold NaN in Q, K and the value input,
and the output is bit for bit the one with zeros there.  One and two tiles, several fibres per tile, heads that share K or do not, narrow rows, the
encoding, lengths that end inside a fibre, at its end and after one token, either kind of value input."""
import numpy as np
import pytest
import torch

import paper_2410_20926_amd as ta
from gpu_util import to_dev, to_host
from paper_2410_20926_amd.workloads import make_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # dims, Hq, Hkv, D, causal, lens, rope base
    ((20, 9, 23), 8, 2, 128, False, (4140, 2071, 1), 10000.0),
    ((5, 7, 3), 4, 4, 64, True, (104, 53, 7), 10000.0),
    ((41, 3), 4, 1, 128, True, (122, 64, 33), None),
    ((6, 50), 3, 3, 64, False, (299, 150, 51), 500.0),
    ((4, 10, 30), 2, 2, 100, False, (1199, 601, 30), None),
]


@pytest.mark.parametrize("vin", [ta.TA_VIN_KV, ta.TA_VIN_O])
@pytest.mark.parametrize("dims,Hq,Hkv,D,causal,lens,rope", CASES)
def test_padding_is_not_read(dims, Hq, Hkv, D, causal, lens, rope, vin):
    N, B = int(np.prod(dims)), len(lens)
    q, k, v = make_inputs(B, N, Hq, Hkv, D, seed=9400 + N + D, dtype="bf16")
    x = q[::-1].copy() if vin == ta.TA_VIN_O else v
    plan = ta.ta_plan_create(B, Hq, Hkv, D, dims, ta.TA_BF16, causal, valid_lens=torch.tensor(lens, dtype=torch.int64, device="cuda"), rope_base=rope)
    for axis in range(len(dims)):
        out = []
        for fill in (0.0, np.nan):
            for t in (q, k, x):
                for b, n in enumerate(lens):
                    t[b, n:] = fill
            o = torch.full((B, N, Hq, D), float("nan"), dtype=torch.bfloat16, device="cuda")
            ta.ta_axis_attn_forward(plan, axis, to_dev(q, "bf16"), to_dev(k, "bf16"), to_dev(x, "bf16"), vin, o)
            torch.cuda.synchronize()
            out.append(to_host(o))
        assert np.isfinite(out[1]).all() and np.array_equal(*out)
        assert all(not out[0][b, n:].any() for b, n in enumerate(lens))


@pytest.mark.parametrize("H,Hkv,rope", [(8, 8, None), (8, 2, 500.0), (6, 2, None)])
@pytest.mark.parametrize("vin", [ta.TA_VIN_KV, ta.TA_VIN_O])
def test_streamed_narrow_rows_give_the_bits_of_cached_ones(H, Hkv, rope, vin):
    """Two tiles, heads of 40 features: a call a little larger than the last-level cache, and each end of it alone."""
    B, n, D, heads = 4, 56, 40, 2 * H + Hkv + (H if vin else Hkv)
    dims = (round(330e6 / (2 * B * n * D * heads)), n)
    gen = torch.Generator(device="cuda").manual_seed(9500 + H)
    q, k, x = (torch.randn((B, dims[0] * n, h, D), generator=gen, device="cuda").bfloat16() for h in (H, Hkv, H if vin else Hkv))

    def hop(form, q, k, x):
        plan = ta.ta_plan_create(q.shape[0], H, Hkv, D, dims, ta.TA_BF16, False, rope_base=rope)
        assert plan.hop_form(1, vin) == (form if vin == ta.TA_VIN_O or H == Hkv else "rows_cached")
        o = torch.full_like(q, float("nan"))
        ta.ta_axis_attn_forward(plan, 1, q, k, x, vin, o)
        return o
    whole = hop("rows_streamed", q, k, x)
    assert torch.isfinite(whole).all()
    for b in (0, B - 1):
        assert torch.equal(whole[b:b + 1], hop("rows_cached", *(t[b:b + 1].contiguous() for t in (q, k, x))))
