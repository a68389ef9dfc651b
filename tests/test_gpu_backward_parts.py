"""The long-axis backward of few fibres is worked out in parts by several workgroups, of many by one workgroup per fibre and key/value head: a batch that fills
the chip gives the bits of its elements alone, at every edge of an eight of tiles, with every mask and the encoding."""
import numpy as np
import pytest
import torch

import paper_2410_20926_amd as ta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vin", [ta.TA_VIN_KV, ta.TA_VIN_O])
@pytest.mark.parametrize("n,fibres,B,H,Hkv,D,causal,window,rope,lens,table", [
    (129, 9, 32, 4, 2, 64, True, 0, None, False, False),   # 576 fibres and key/value heads, 18 alone; five tiles, the last of one row
    (256, 8, 32, 3, 3, 128, True, 0, None, True, False),   # eight tiles
    (257, 8, 32, 2, 2, 40, False, 0, 500.0, False, False), # eight and a row
    (300, 6, 40, 4, 2, 100, True, 40, None, False, False), # a band: parts that see few others
    (520, 2, 130, 4, 2, 64, True, 0, 10000.0, True, True),
    (330, 3, 96, 6, 2, 128, False, 100, None, True, False),
])
def test_parts_give_the_bits_of_the_whole(n, fibres, B, H, Hkv, D, causal, window, rope, lens, table, vin):
    dims, N, gen = (n, fibres), n * fibres, torch.Generator(device="cuda").manual_seed(n + D)
    q, x, g = (torch.randn((B, N, h, D), generator=gen, device="cuda").bfloat16() for h in (H, H if vin else Hkv, H))
    k = torch.randn((B, N, Hkv, D), generator=gen, device="cuda").bfloat16()
    ends = torch.randint(N // 3, N + 1, (B,), generator=gen, device="cuda", dtype=torch.int64)
    mask = (np.random.default_rng(n).random((n, n)) < 0.6) | np.eye(n, dtype=bool)
    packed = torch.from_numpy(ta.pack_axis_mask(mask)).cuda()

    def hop(b):
        kw = dict(window=(window, 0), rope_base=rope, valid_lens=ends[b].contiguous() if lens else None, axis_masks=[packed if table else None, None])
        rows = [t[b].contiguous() for t in (q, k, x, g)]
        plan = ta.ta_plan_create(rows[0].shape[0], H, Hkv, D, dims, ta.TA_BF16, causal, **kw)
        assert plan.hop_function(0, vin, True) == "mfma_bwd_long_kernel"
        dq, dk, dx = (torch.full_like(t, 0.25) for t in rows[:3])
        for accumulate in (False, True):
            ta.ta_axis_attn_backward(plan, 0, rows[0], rows[1], rows[2], vin, rows[3], dx, dq, dk, accumulate)
        return dq, dk, dx
    whole = hop(slice(None))
    assert all(torch.isfinite(t).all() for t in whole)
    for b in (0, B // 2, B - 1):
        assert all(torch.equal(t[b:b + 1], y) for t, y in zip(whole, hop(slice(b, b + 1)))), b
