"""The long-axis forward whose workgroup works in two phases (eight query tiles, enough of them for every CU), at its edges: axes that end
one row after and before a tile, a block and a workgroup, single heads and groups of four, bands, padding, bit tables, narrow rows.  A part of
the same call on its own has too few workgroups for it and runs four tiles in step, with the same arithmetic in the same order: same bits.
One part is compared with 64 bits."""
import math

import pytest
import torch

import paper_2410_20926_amd as ta
from gpu_util import TOL
from paper_2410_20926_amd.workloads import make_inputs

pytestmark = pytest.mark.gpu


FOUR, PHASES = "four_tiles_in_step", "eight_tiles_in_phases"


def call(q, k, v, n, causal, window, valid, table=None, form=None):
    B, _, H, D = q.shape
    plan = ta.ta_plan_create(B, H, k.shape[2], D, (n,), ta.TA_BF16, causal, window=(window,), valid_len=valid, axis_masks=[table])
    assert form in (None, plan.hop_form(0, ta.TA_VIN_KV))
    o = torch.full_like(q, 7.0)
    ta.ta_axis_attn_forward(plan, 0, q, k, v, ta.TA_VIN_KV, o)
    return o


def band_table(n, window):
    a, c = torch.arange(n)[:, None], torch.arange(n)[None, :]
    return torch.from_numpy(ta.pack_axis_mask(((a - c).abs() < window).numpy())).cuda()


@pytest.mark.parametrize("n,B,H,Hkv,D,causal,window,valid,tabled", [
    (2048, 4, 8, 8, 64, True, 0, 0, False),
    (2047, 4, 8, 8, 128, True, 0, 0, False),                # 256 workgroups: one full round of them
    (1029, 12, 8, 8, 64, False, 0, 1025, False),            # 480, and 1,020: the last round is nearly full
    (1025, 15, 16, 4, 128, False, 0, 0, False),
    (2049, 4, 8, 8, 128, True, 0, 0, False),
    (2111, 30, 1, 1, 128, False, 700, 0, False),            # (short windows and tables: four tiles in the whole call too)
    (2111, 30, 1, 1, 64, False, 700, 0, True),
    (2111, 30, 1, 1, 128, False, 1000, 0, False),
    (2080, 30, 1, 1, 64, True, 2060, 0, False),
    (2080, 2, 16, 4, 128, True, 0, 1500, False),            # four heads that share K and the values side by side
    (2303, 2, 16, 4, 64, False, 90, 2301, False),
    (2303, 2, 16, 4, 64, False, 1100, 2301, False),
    (4097, 4, 4, 4, 100, True, 0, 0, False),
    (4128, 4, 4, 4, 40, False, 1000, 4000, False),
])
def test_phases_give_the_bits_of_four_tiles_in_step(n, B, H, Hkv, D, causal, window, valid, tabled):
    q, k, v = (torch.from_numpy(x).cuda().to(torch.bfloat16) for x in make_inputs(B, n, H, Hkv, D, seed=890 + n + D, dtype="bf16"))
    G, rows = H // Hkv, 256 // (4 if H // Hkv == 4 else 1)
    blocks = (n + rows - 1) // rows
    assert B * Hkv * blocks >= 256 > blocks                # the whole call may run in phases, a part of it not
    table = band_table(n, window) if tabled else None
    whole = call(q, k, v, n, causal, 0 if tabled else window, valid, table, FOUR if window in (90, 700) else PHASES)
    for b in range(0, B, 3):
        for g in range(Hkv):
            at = slice(b, b + 1), slice(None), slice(g * G, (g + 1) * G)
            kv = slice(b, b + 1), slice(None), slice(g, g + 1)
            part = call(q[at].contiguous(), k[kv].contiguous(), v[kv].contiguous(), n, causal, window, valid, None, FOUR)
            assert torch.equal(part, whole[at]), (b, g)
    a, c = torch.arange(n, device="cuda")[:, None], torch.arange(n, device="cuda")[None, :]
    live = valid or n
    see = (a < live) & (c < live) & ((c <= a) if causal else (c == c)) & (((a - c).abs() < window) if window else (c == c))
    Q, K, V = (x[0, :, 0].double() for x in (q, k, v))
    p = torch.softmax((Q @ K.t() / math.sqrt(D)).masked_fill(~see, -math.inf), -1).nan_to_num(0.0)
    err = (whole[0, :, 0].double() - p @ V).abs().max().item()
    assert err <= TOL["bf16"], f"{err:.3e}"


@pytest.mark.parametrize("n,D,causal,window,valid", [(2080, 128, True, 0, 2080), (2100, 64, False, 300, 1700), (3100, 64, False, 1100, 2700)])
def test_values_out_of_reach_stay_out(n, D, causal, window, valid):
    """An infinity in a value row reaches only the query tiles some row of which sees a key of its tile of 32, padding reaches no row."""
    B, H = 4, 8
    q, k, v = (torch.from_numpy(x).cuda().to(torch.bfloat16) for x in make_inputs(B, n, H, H, D, seed=893, dtype="bf16"))
    clean = call(q, k, v, n, causal, window, valid, None, FOUR if window == 300 else PHASES)
    assert (clean[:, valid:] == 0).all()
    bad_k, bad_v = k.clone(), v.clone()
    bad_k[:, valid:], bad_v[:, (valid + 31) // 32 * 32:] = float("nan"), float("inf")
    assert torch.equal(call(q, bad_k, bad_v, n, causal, window, valid), clean)
    for c in (45, valid // 2, valid - 1):
        bad_v = v.clone()
        bad_v[:, c] = float("inf")
        got = call(q, k, bad_v, n, causal, window, valid)
        c0 = c // 32 * 32
        for a0 in range(0, valid, 32):
            a1 = a0 + 31
            if (causal and c0 > a1) or (window and (c0 - a1 >= window or a0 - (c0 + 31) >= window)):
                assert torch.equal(got[:, a0:a1 + 1], clean[:, a0:a1 + 1]), (c, a0)
        assert not torch.isfinite(got[0, c]).any()


@pytest.mark.parametrize("vin", [ta.TA_VIN_KV, ta.TA_VIN_O])
@pytest.mark.parametrize("dims,axis,B,H,Hkv,D,causal,window,valid", [
    ((2056, 3), 0, 2, 8, 8, 128, True, 0, 0),               # 8 rows past a workgroup: one wave works, on a quarter of a tile, seven fetch
    ((3, 2200), 1, 2, 8, 8, 64, True, 0, 0),                # five tiles, the last of 24 rows
    ((2200, 3), 0, 2, 16, 4, 64, False, 2100, 0),           # groups of four: two tiles per workgroup
    ((2, 4100, 2), 1, 1, 4, 4, 100, True, 0, 0),            # several fibres, rows apart and narrow
    ((4100, 3), 0, 2, 4, 4, 40, False, 0, 9000),            # padding begins inside the axis
])
def test_last_workgroup_and_rows_apart(dims, axis, B, H, Hkv, D, causal, window, valid, vin):
    """Axes that end a few rows into a workgroup, with rows that are not neighbours in memory and several fibres: same bits as four tiles in step."""
    N, n = math.prod(dims), dims[axis]
    q, k, v = (torch.from_numpy(x).cuda().to(torch.bfloat16) for x in make_inputs(B, N, H, Hkv, D, seed=896 + N + D, dtype="bf16"))
    x = q.flip(0, 1).contiguous() if vin == ta.TA_VIN_O else v
    G = H // Hkv

    def hop(q, k, x, form):
        plan = ta.ta_plan_create(q.shape[0], q.shape[2], k.shape[2], D, dims, ta.TA_BF16, causal, valid_len=valid,
                                 window=tuple(window if a == axis else 0 for a in range(len(dims))))
        assert plan.hop_form(axis, vin) == form
        o = torch.full_like(q, 7.0)
        ta.ta_axis_attn_forward(plan, axis, q, k, x, vin, o)
        return o
    whole = hop(q, k, x, PHASES)
    for b in range(B):
        for g in range(0, Hkv, 3):
            at = slice(b, b + 1), slice(None), slice(g * G, (g + 1) * G)
            kv = slice(b, b + 1), slice(None), slice(g, g + 1)
            assert torch.equal(hop(q[at].contiguous(), k[kv].contiguous(), x[at if vin == ta.TA_VIN_O else kv].contiguous(), FOUR), whole[at]), (b, g)
    if valid:
        assert not whole[:, valid:].any()
    fibre = torch.arange(N, device="cuda").view(dims).movedim(axis, -1).reshape(-1, n)[1]    # the second fibre of the last sequence's first head
    a, c = torch.arange(n, device="cuda")[:, None], torch.arange(n, device="cuda")[None, :]
    live = fibre < (valid or N)
    see = live[:, None] & live[None, :] & ((c <= a) if causal else (c == c)) & (((a - c).abs() < window) if window else (c == c))
    Q, K, X = (t[-1, fibre, 0].double() for t in (q, k, x))
    p = torch.softmax((Q @ K.t() / math.sqrt(D)).masked_fill(~see, -math.inf), -1).nan_to_num(0.0)
    err = (whole[-1, fibre, 0].double() - p @ X).abs().max().item()
    assert err <= TOL["bf16"], f"{err:.3e}"
