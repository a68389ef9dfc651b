"""Rows narrower than their tile, by where they start: whole 16-byte units on 16-byte boundaries, 8 bytes into one for every other head, or for every
other token (an odd number of heads of 100).  A head among others gives the bits of that head alone, forward and backward, on one tile, two, and three,
in grids of every remainder by eight; the oracle is met by the other tests of these kernels."""
import pytest
import torch

import paper_2410_20926_amd as ta

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [8, 12, 36, 40, 60, 68, 96, 100, 124])
@pytest.mark.parametrize("n,fibres,B,H,Hkv", [
    (32, 5, 2, 3, 3),                                      # one tile: 15 workgroups per sequence, rows 8 bytes off on every other token where D % 8 = 4
    (9, 41, 1, 8, 8),                                      # three fibres per tile, the last tile not full; two heads per workgroup in the backward's pairs
    (31, 37, 2, 8, 2),                                     # a group of four
    (33, 3, 1, 4, 4),                                      # two tiles, the second of one row
    (64, 2, 2, 5, 1),                                      # a group of five
    (96, 3, 1, 8, 2),
    (200, 2, 1, 4, 2),
    (70, 5, 1, 8, 2),                                      # the streaming forward of groups of four, all query tiles of a fibre in one workgroup
    (190, 3, 1, 4, 1),                                     # and one per workgroup, on the first hop
    (32, 131, 1, 6, 6),                                    # enough workgroups to be put in order, no multiple of eight: 262 forward, 786 backward
    (17, 299, 1, 8, 2),                                    # 598
])
def test_a_head_among_others_gives_the_bits_of_the_head_alone(D, n, fibres, B, H, Hkv):
    gen, N, G = torch.Generator(device="cuda").manual_seed(100 * D + n), n * fibres, H // Hkv
    q, x, g = (torch.randn((B, N, H, D), generator=gen, device="cuda").bfloat16() for _ in range(3))
    k = torch.randn((B, N, Hkv, D), generator=gen, device="cuda").bfloat16()
    for dims, axis in (((n, fibres), 0), ((fibres, n), 1)):
        def hops(q, k, x, g):
            plan = ta.ta_plan_create(B, q.shape[2], k.shape[2], D, dims, ta.TA_BF16, True)
            o, o1, (dq, dk, dx) = torch.full_like(q, float("nan")), torch.full_like(q, float("nan")), (torch.full_like(t, 0.5) for t in (q, k, x))
            ta.ta_axis_attn_forward(plan, axis, q, k, x, ta.TA_VIN_O, o)
            ta.ta_axis_attn_forward(plan, axis, q, k, k, ta.TA_VIN_KV, o1)
            for accumulate in (False, True):
                ta.ta_axis_attn_backward(plan, axis, q, k, x, ta.TA_VIN_O, g, dx, dq, dk, accumulate)
            return torch.stack((o, o1)), dq, dx, dk
        whole = hops(q, k, x, g)
        assert all(torch.isfinite(t).all() for t in whole)
        for j in {0, Hkv // 2, Hkv - 1}:
            heads = slice(j * G, (j + 1) * G)
            part = hops(*(t.contiguous() for t in (q[:, :, heads], k[:, :, j:j + 1], x[:, :, heads], g[:, :, heads])))
            assert all(torch.equal(t[..., heads, :], y) for t, y in zip(whole[:3], part)) and torch.equal(whole[3][:, :, j:j + 1], part[3]), (dims, j)


@pytest.mark.parametrize("D", [12, 40, 60])
@pytest.mark.parametrize("dims,H,Hkv", [((3, 12, 7), 3, 3), ((2, 16, 8), 8, 2), ((2, 28, 4), 5, 5)])
def test_small_slabs_give_the_bits_of_their_heads_alone(D, dims, H, Hkv):
    gen, N, G = torch.Generator(device="cuda").manual_seed(D + H), dims[0] * dims[1] * dims[2], H // Hkv
    q = torch.randn((2, N, H, D), generator=gen, device="cuda").bfloat16()
    k, v = (torch.randn((2, N, Hkv, D), generator=gen, device="cuda").bfloat16() for _ in range(2))

    def forward(q, k, v):
        plan = ta.ta_plan_create(2, q.shape[2], k.shape[2], D, dims, ta.TA_BF16, True)
        assert plan.small_pair_position() == 1
        o, ws = torch.full_like(q, float("nan")), torch.empty(max(plan.workspace_bytes(False), 256), dtype=torch.uint8, device="cuda")
        ta.ta_multihop_forward(plan, q, k, v, o, ws, plan.workspace_bytes(False))
        return o
    whole = forward(q, k, v)
    assert torch.isfinite(whole).all()
    for j in range(Hkv):
        assert torch.equal(whole[:, :, j * G:(j + 1) * G], forward(*(t.contiguous() for t in (q[:, :, j * G:(j + 1) * G], k[:, :, j:j + 1], v[:, :, j:j + 1]))))


@pytest.mark.parametrize("F,H,Hkv,n,D", [
    (3328, 3, 3, 33, 40),                                  # 9,984 (fibre, head) pairs: the first size whose workgroups take four of them
    (3327, 3, 3, 33, 36),                                  # one fibre less: as many workgroups as are resident
    (2816, 4, 4, 33, 100),                                 # the same in 128-wide tiles, 11,264 pairs
    (2815, 4, 4, 33, 68),
    (4099, 3, 3, 64, 100),                                 # a last workgroup of fewer, and some of five
    (3073, 8, 4, 40, 12),                                  # groups of two heads
])
def test_two_tile_backward_in_short_shares_gives_the_bits_of_a_few_fibres(F, H, Hkv, n, D):
    gen = torch.Generator(device="cuda").manual_seed(F + D)
    q, x, g = (torch.randn((1, F * n, H, D), generator=gen, device="cuda").bfloat16() for _ in range(3))
    k = torch.randn((1, F * n, Hkv, D), generator=gen, device="cuda").bfloat16()

    def hop(vin, q, k, x, g):
        plan = ta.ta_plan_create(1, H, Hkv, D, (q.shape[1] // n, n), ta.TA_BF16, True)
        dq, dk, dx = (torch.full_like(t, 0.5) for t in (q, k, x))
        ta.ta_axis_attn_backward(plan, 1, q, k, x, vin, g, dx, dq, dk, True)
        return dq, dk, dx
    for vin, value in ((ta.TA_VIN_O, x), (ta.TA_VIN_KV, k)):
        whole = hop(vin, q, k, value, g)
        assert all(torch.isfinite(t).all() for t in whole)
        for f in (0, F // 2, F - 5):
            part = slice(f * n, (f + 5) * n)
            for a, b in zip(whole, hop(vin, *(t[:, part].clone() for t in (q, k, value, g)))):
                assert torch.equal(a[:, part], b)


@pytest.mark.parametrize("rope", [None, 10000.0])
@pytest.mark.parametrize("vin", [ta.TA_VIN_KV, ta.TA_VIN_O])
@pytest.mark.parametrize("n,H,Hkv,D", [(32, 8, 8, 100), (32, 16, 4, 96), (50, 8, 8, 96), (50, 16, 4, 100)])
def test_streamed_wide_rows_give_the_bits_of_cached_ones(n, H, Hkv, D, vin, rope):
    """One and two tiles, 128-wide: a forward call a little larger than the last-level cache is streamed, elements of its batch alone are cached, a few of their
    fibres, which the other tests compare with the oracle, streamed again."""
    B, heads = 5, 2 * H + Hkv + (H if vin else Hkv)
    fibres, gen = round(340e6 / (2 * B * n * D * heads)), torch.Generator(device="cuda").manual_seed(n + D)
    q, k, x = (torch.randn((B, fibres * n, h, D), generator=gen, device="cuda").bfloat16() for h in (H, Hkv, H if vin else Hkv))

    def hop(form, q, k, x):
        plan = ta.ta_plan_create(q.shape[0], H, Hkv, D, (q.shape[1] // n, n), ta.TA_BF16, True, rope_base=rope)
        assert plan.hop_form(1, vin) == form and plan.hop_function(1, vin) == ("mfma_fwd_kernel" if H == Hkv else "mfma_fwd_shared_kernel")
        o = torch.full_like(q, float("nan"))
        ta.ta_axis_attn_forward(plan, 1, q, k, x, vin, o)
        return o
    whole = hop("rows_streamed", q, k, x)
    assert torch.isfinite(whole).all()
    for b in (0, 2, B - 1):
        cached = hop("rows_cached", *(t[b:b + 1].contiguous() for t in (q, k, x)))
        few = hop("rows_streamed", *(t[b:b + 1, :7 * n].contiguous() for t in (q, k, x)))
        assert torch.equal(whole[b:b + 1], cached) and torch.equal(cached[:, :7 * n], few)


@pytest.mark.parametrize("D,n,H", [(36, 10, 16), (28, 32, 24), (60, 32, 12), (48, 9, 16), (20, 31, 16)])
def test_rows_far_apart_give_the_bits_of_rows_nearby(D, n, H):
    """Rows of a fibre 2 MB apart, in a call that leaves the last-level cache (and one that does not): the forward of one tile by heads alone, whose rows are nearer."""
    fibres = -(-(2 << 20) // (H * D * 2)) + 3
    for B in (1, -(-290000000 // (8 * n * fibres * H * D))):
        gen = torch.Generator(device="cuda").manual_seed(D + n)
        q, k, x = (torch.randn((B, n * fibres, H, D), generator=gen, device="cuda").bfloat16() for _ in range(3))

        def hop(*rows):
            plan = ta.ta_plan_create(rows[0].shape[0], rows[0].shape[2], rows[0].shape[2], D, (n, fibres), ta.TA_BF16, True)
            assert plan.hop_function(0, ta.TA_VIN_O) == "mfma_fwd_kernel"
            o = torch.full_like(rows[0], float("nan"))
            ta.ta_axis_attn_forward(plan, 0, *rows[:2], rows[2], ta.TA_VIN_O, o)
            return o
        whole = hop(q, k, x)
        assert torch.isfinite(whole).all()
        for b in {0, B // 2, B - 1}:
            for h in (0, 1, H // 2, H - 1):
                assert torch.equal(whole[b:b + 1, :, h:h + 1], hop(*(t[b:b + 1, :, h:h + 1].contiguous() for t in (q, k, x)))), (B, b, h)
