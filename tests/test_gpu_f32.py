"""GPU parity of the fp32 matrix kernels at the sizes where they can go wrong: one fibre and many per tile,
axes on both sides of a tile, row widths on both sides of the 32-, 64- and 128-wide tiles, grouped heads, every mask, the
encoding; and a fault (infinity) in one fibre that must not reach the fibres that share its tile."""
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
    # dims, B, Hq, Hkv, D, causal, window, valid_len, rope base
    ((1, 5, 16), 1, 3, 3, 64, False, None, None, None),        # unit axis: 16 fibres per tile; a last tile that is part full
    ((17, 31), 2, 2, 1, 32, True, None, None, None),           # one fibre per tile
    ((32, 33), 1, 4, 2, 36, True, (0, 9), 1000, None),         # a whole tile; one row more than a tile
    ((9, 64), 1, 1, 1, 128, False, None, None, None),
    ((65, 3), 1, 6, 2, 100, True, None, 150, 200.0),
    ((2, 130), 2, 2, 2, 68, False, (0, 40), None, None),
    ((3, 2, 200), 1, 2, 1, 4, True, None, None, 100.0),        # the narrowest row
    ((7, 3), 3, 8, 2, 12, False, (2, 0), 17, 100.0),
]


@pytest.mark.parametrize("dims,B,Hq,Hkv,D,causal,window,valid_len,rope", CASES)
def test_fp32_hops_match_oracle(dims, B, Hq, Hkv, D, causal, window, valid_len, rope):
    N = int(np.prod(dims))
    q, k, v, d_o = make_inputs(B, N, Hq, Hkv, D, seed=8100 + N + D, dtype="f32", with_grad=True)
    kw = dict(window=window, rope_base=rope)
    got, plan, dev = multihop_forward(q, k, v, dims, "f32", causal, save=True, valid_len=valid_len or 0, **kw)
    ref = orc.tensorized_attention_forward(q, k, v, dims, causal, valid_len=valid_len, **kw)
    err = np.abs(got - ref).max()
    assert np.isfinite(got).all() and err <= TOL["f32"], f"forward: {err:.3e}"
    for axis, n in enumerate(dims):
        assert [plan.hop_function(axis, ta.TA_VIN_O, b) for b in (False, True)] == (["f32_fwd_kernel", "f32_bwd_kernel"] if n <= 32 else ["f32_fwd_long_kernel", "f32_bwd_long_kernel"])
    grads = multihop_backward(plan, dev, d_o, "f32")
    check_backward(grads, q, k, v, d_o, dims, causal, "f32", valid_len=valid_len, **kw)


@pytest.mark.parametrize("n,D", [(8, 64), (5, 128), (4, 32)])
def test_a_fault_in_one_fibre_stays_there(n, D):
    """Fibres of the last axis share tiles: an infinity or NaN in one fibre's rows of any input leaves the results of
    every other fibre what they are without it (same bits: the same sums in the same order, with zeros beside them)."""
    dims, H = (9, n), 2
    N = 9 * n
    q, k, v, d_o = (torch.from_numpy(x).cuda() for x in make_inputs(1, N, H, H, D, seed=811, dtype="f32", with_grad=True))
    plan = ta.ta_plan_create(1, H, H, D, dims, ta.TA_F32, False)

    def run(q, k, v, g):
        o, dx, dq, dk = (torch.zeros_like(q) for _ in range(4))
        ta.ta_axis_attn_forward(plan, 1, q, k, v, ta.TA_VIN_O, o)
        ta.ta_axis_attn_backward(plan, 1, q, k, v, ta.TA_VIN_O, g, dx, dq, dk, False)
        return [t.cpu() for t in (o, dx, dq, dk)]

    clean = run(q, k, v, d_o)
    bad = [x.clone() for x in (q, k, v, d_o)]
    bad[2][0, n + 1, :, 3] = float("inf")                      # fibre 1
    bad[3][0, 2 * n, :, 0] = float("nan")                      # fibre 2
    bad[0][0, 4 * n + 1, :, 2] = float("nan")                  # fibre 4
    bad[1][0, 6 * n, :, 1] = float("inf")                      # fibre 6
    got = run(*bad)
    others = [t for t in range(N) if t // n not in (1, 2, 4, 6)]
    for a, b in zip(clean, got):
        assert torch.equal(a[:, others], b[:, others])
    for result, fibre in ((0, 1), (1, 2), (0, 4), (2, 4), (0, 6), (3, 6)):
        assert not torch.isfinite(got[result][:, fibre * n:(fibre + 1) * n]).all()


@pytest.mark.parametrize("n,D,causal,window,valid", [
    (6, 64, False, 0, 20), (12, 128, True, 0, 17), (24, 64, False, 0, 40), (30, 100, True, 5, 70), (100, 64, False, 0, 37), (100, 128, True, 0, 150),
    (130, 36, False, 9, 300), (65, 128, False, 0, 64)])
def test_values_that_no_row_sees_reach_none(n, D, causal, window, valid):
    """Padding is never attended to and gives zeros, whatever its rows hold: with infinities and NaN in the padding of K and the
    values, every output is what it is with zeros there (same bits).  The same for keys that a row does not see for any other reason:
    an infinity in one value row reaches the rows that see it, and no others."""
    for dims, axis in (((4, n), 1), ((n, 3), 0)):
        N, H = int(np.prod(dims)), 2
        q, k, v = (torch.from_numpy(x).cuda() for x in make_inputs(1, N, H, H, D, seed=812, dtype="f32"))
        valid = min(valid, N)
        plan = ta.ta_plan_create(1, H, H, D, dims, ta.TA_F32, causal, window=tuple(window if i == axis else 0 for i in range(2)), valid_len=valid)

        def run(k, v):
            o = torch.full_like(q, 7.0)
            ta.ta_axis_attn_forward(plan, axis, q, k, v, ta.TA_VIN_O, o)
            return o.cpu()

        k[:, valid:], v[:, valid:] = 0.0, 0.0
        clean = run(k, v)
        bad_k, bad_v = k.clone(), v.clone()
        bad_k[:, valid:], bad_v[:, valid:] = float("nan"), float("inf")
        bad_v[:, valid::2] = float("nan")
        got = run(bad_k, bad_v)
        assert torch.equal(got, clean) and (got[:, valid:] == 0).all()

        stride = N // n if axis == 0 else 1
        c = min(n - 1, (valid - 1) // stride if axis == 0 else valid - 1) // 2      # a real key of the first fibre
        bad_v = v.clone()
        bad_v[:, c * stride, :, 1] = float("inf")
        got = run(k, bad_v)
        for a in range(n):
            sees = a * stride < valid and (not causal or c <= a) and (not window or abs(a - c) < window)
            row, ref = got[0, a * stride], clean[0, a * stride]
            assert torch.equal(row[:, 0], ref[:, 0]) or sees            # (another order of sums where it is seen)
            assert torch.isinf(row[:, 1]).all() if sees else torch.equal(row, ref)


def chain(a, b, steps):
    """fp32 sum over `steps` of outer products a(i) * b(i), one multiply-add after the other (products exact, every sum rounded once)."""
    acc = np.float32(0)
    for i in steps:
        acc = (a(i).astype(np.float64) * b(i) + acc).astype(np.float32)
    return acc


def halves(x, y):
    """x [F, n, D] times y^T, every row of products summed in two halves: what the vector kernels do."""
    D = x.shape[-1]
    return sum(chain(lambda d: x[:, :, None, d], lambda d: y[:, None, :, d], range(i * D // 2, (i + 1) * D // 2)) for i in (0, 1))


@pytest.mark.parametrize("n,D,fibres", [(16, 64, 96), (11, 128, 96), (32, 128, 48), (24, 100, 48), (64, 128, 24), (40, 64, 24)])
def test_scores_lose_no_more_than_sums_over_half_rows(n, D, fibres):
    """Rounding error (2-norm against 64 bits) of one hop and its gradients, against the same hop in fp32 with scores and dP summed over
    half rows: a longer chain of sums per score, e.g. one over the whole row, gives a larger error (1.3 times and more in o)."""
    N = n * fibres
    q, k, v, g = make_inputs(1, N, 1, 1, D, seed=8200 + n + D, dtype="f32", with_grad=True)
    f = [x.reshape(fibres, n, D) for x in (q, k, v, g)]
    scale = np.float32(1 / np.sqrt(D))

    s = halves(f[0], f[1]) * scale
    w = np.exp(s - s.max(-1, keepdims=True))
    inv = np.float32(1) / w.sum(-1, keepdims=True)
    p, dp = w * inv, halves(f[3], f[2])
    ds = p * (dp - (p * dp).sum(-1, keepdims=True))
    low = [chain(lambda c: w[:, :, c, None], lambda c: f[2][:, c, None], range(n)) * inv,
           chain(lambda c: p[:, c, :, None], lambda c: f[3][:, c, None], range(n)),
           chain(lambda c: ds[:, :, c, None], lambda c: f[1][:, c, None], range(n)) * scale]

    q64, k64, v64, g64 = (x.astype(np.float64) for x in f)
    s = q64 @ k64.swapaxes(1, 2) / np.sqrt(D)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    dp = g64 @ v64.swapaxes(1, 2)
    ds = p * (dp - (p * dp).sum(-1, keepdims=True))
    exact = [p @ v64, p.swapaxes(1, 2) @ g64, ds @ k64 / np.sqrt(D)]

    dev = [torch.from_numpy(x).cuda() for x in (q, k, v, g)]
    plan = ta.ta_plan_create(1, 1, 1, D, (fibres, n), ta.TA_F32, False)
    o, dx, dq, dk = (torch.zeros_like(dev[0]) for _ in range(4))
    ta.ta_axis_attn_forward(plan, 1, *dev[:3], ta.TA_VIN_O, o)
    ta.ta_axis_attn_backward(plan, 1, *dev[:3], ta.TA_VIN_O, dev[3], dx, dq, dk, False)
    for name, got, ref, low_one in zip(("o", "dx", "dq"), (o, dx, dq), exact, low):
        got = got.cpu().numpy().reshape(fibres, n, D).astype(np.float64)
        size = np.linalg.norm(ref)
        err, bound = np.linalg.norm(got - ref) / size, np.linalg.norm(low_one - ref) / size
        assert err <= bound, f"{name}: {err:.3e}, with half rows {bound:.3e}"


@pytest.mark.parametrize("n", [7, 16, 25, 32, 45])
def test_turned_rows_are_rounded_once(n):
    """With an upstream gradient on one row a of a fibre only, dK of position 0 (which is not turned back) is a multiple of the turned
    query row a: two roundings, one of the turned row and one of the product, each 2.5e-8 in the 2-norm on average (an error evenly
    spread up to half a unit in the last place of mantissas of every size), 3.5e-8 together; a row turned in fp32 arithmetic
    carries 4.2e-8 and gives 4.9e-8."""
    H, D, fibres = 4, 64, 64
    N = n * fibres
    q, k, v, g = make_inputs(1, N, H, H, D, seed=8250 + n, dtype="f32", with_grad=True)
    rows = np.arange(fibres) % (n - 1) + 1                     # the row of each fibre that has a gradient
    keep = np.zeros((fibres, n, 1, 1), np.float32)
    keep[np.arange(fibres), rows] = 1
    g = (g.reshape(fibres, n, H, D) * keep).reshape(1, N, H, D)
    dev = [torch.from_numpy(x).cuda() for x in (q, k, v, g)]
    plan = ta.ta_plan_create(1, H, H, D, (fibres, n), ta.TA_F32, False, rope_base=8192.0)      # (a base whose logarithm, kept in fp32, is exact)
    dx, dq, dk = (torch.zeros_like(dev[0]) for _ in range(3))
    ta.ta_axis_attn_backward(plan, 1, *dev[:3], ta.TA_VIN_O, dev[3], dx, dq, dk, False)
    got = dk.cpu().numpy().astype(np.float64).reshape(fibres, n, H, D)[:, 0]
    x = q.astype(np.float64).reshape(fibres, n, H, D)[np.arange(fibres), rows]
    ang = rows[:, None, None] * 8192.0 ** (-np.arange(0, D, 2) / D)
    turned = np.empty_like(x)
    turned[..., 0::2] = x[..., 0::2] * np.cos(ang) - x[..., 1::2] * np.sin(ang)
    turned[..., 1::2] = x[..., 0::2] * np.sin(ang) + x[..., 1::2] * np.cos(ang)
    turned *= (got * turned).sum(-1, keepdims=True) / (turned * turned).sum(-1, keepdims=True)
    err = np.sqrt((((got - turned) ** 2).sum(-1) / (turned ** 2).sum(-1)).mean())
    assert err <= 1.15 * 3.5e-8, f"{err:.3e}"


@pytest.mark.parametrize("n,fibres", [(12, 96), (32, 48), (70, 24)])
def test_weights_lose_no_more_than_expf_of_scaled_scores(n, fibres):
    """Whole-numbered queries and keys: every score is exact, and the error left is that of the softmax and of the sums after it.  The
    scale is one whose product with log2(e) loses 7e-8 of itself when it is rounded to fp32."""
    D, scale = 64, np.float32(0.1813800036907196)
    N = n * fibres
    rng = np.random.default_rng(n)
    q, k = (rng.integers(-2, 3, (1, N, 1, D)).astype(np.float32) for _ in range(2))
    _, _, v, g = make_inputs(1, N, 1, 1, D, seed=8270 + n, dtype="f32", with_grad=True)
    f = [x.reshape(fibres, n, D) for x in (q, k, v, g)]

    s = (f[0] @ f[1].swapaxes(1, 2)) * scale
    w = np.exp(s - s.max(-1, keepdims=True))
    inv = np.float32(1) / w.sum(-1, keepdims=True)
    low = [chain(lambda c: w[:, :, c, None], lambda c: f[2][:, c, None], range(n)) * inv,
           chain(lambda c: (w * inv)[:, c, :, None], lambda c: f[3][:, c, None], range(n))]
    q64, k64, v64, g64 = (x.astype(np.float64) for x in f)
    s = q64 @ k64.swapaxes(1, 2) * np.float64(scale)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)

    dev = [torch.from_numpy(x).cuda() for x in (q, k, v, g)]
    plan = ta.ta_plan_create(1, 1, 1, D, (fibres, n), ta.TA_F32, False, scale=float(scale))
    o, dx, dq, dk = (torch.zeros_like(dev[0]) for _ in range(4))
    ta.ta_axis_attn_forward(plan, 1, *dev[:3], ta.TA_VIN_O, o)
    ta.ta_axis_attn_backward(plan, 1, *dev[:3], ta.TA_VIN_O, dev[3], dx, dq, dk, False)
    for name, got, ref, low_one in zip(("o", "dx"), (o, dx), (p @ v64, p.swapaxes(1, 2) @ g64), low):
        got = got.cpu().numpy().reshape(fibres, n, D).astype(np.float64)
        size = np.linalg.norm(ref)
        err, bound = np.linalg.norm(got - ref) / size, np.linalg.norm(low_one - ref) / size
        assert err <= bound, f"{name}: {err:.3e}, with expf {bound:.3e}"


def test_scores_at_the_ends_of_the_range():
    """A score of -inf weighs nothing, a row of such scores gives zeros, and NaN and +inf scores give NaN in their own row only."""
    D, n = 64, 40
    for rows in (n, 16, 24):                                   # streaming, and tiles of 16 and of 32 rows
        q, k, v = (torch.ones(1, rows, 1, D, device="cuda") for _ in range(3))
        v[0, :, 0, :] = torch.arange(rows, device="cuda", dtype=torch.float32)[:, None]
        q[0, 1], q[0, 2], q[0, 3] = -3e38, 3e38, float("nan")
        k[0, 0] = 2.0                                          # scores of row 0: key 0 ahead
        plan = ta.ta_plan_create(1, 1, 1, D, (rows,), ta.TA_F32, False)
        o = torch.zeros_like(q)
        ta.ta_axis_attn_forward(plan, 0, q, k, v, ta.TA_VIN_O, o)
        o = o.cpu()
        assert (o[0, 1] == 0).all() and torch.isnan(o[0, 2:4]).all()
        w = torch.exp((k[0, :, 0].double() @ q[0, :, 0].double().T / 8).T.cpu())
        ref = (w / w.sum(-1, keepdim=True)) @ v[0, :, 0].double().cpu()
        keep = [r for r in range(rows) if r not in (1, 2, 3)]
        assert (o[0, keep, 0] - ref[keep]).abs().max() <= TOL["f32"] * rows      # values up to `rows`


def test_more_workgroups_than_one_grid_dimension_holds():
    """16,777,280 fibres of an odd-width head, one workgroup each: a one-dimensional grid of 256 lanes per workgroup ends at 2^24."""
    H, D, dims = 8, 2, (2097160, 2)
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, g = (torch.randn((1, dims[0] * 2, H, D), generator=gen, device="cuda") for _ in range(4))
    plan = ta.ta_plan_create(1, H, H, D, dims, ta.TA_F32, False)
    o, dx, dq, dk = (torch.full_like(q, 7.0) for _ in range(4))
    ta.ta_axis_attn_forward(plan, 1, q, k, v, ta.TA_VIN_O, o)
    ta.ta_axis_attn_backward(plan, 1, q, k, v, ta.TA_VIN_O, g, dx, dq, dk, False)
    f = [x.view(dims[0], 2, H, D).transpose(1, 2).double() for x in (q, k, v, g)]         # [fibre, head, position, feature]
    p = torch.softmax((f[0][:, :, :, None] * f[1][:, :, None]).sum(-1) / D ** 0.5, -1)    # [fibre, head, row, key]
    dp = (f[3][:, :, :, None] * f[2][:, :, None]).sum(-1)
    ds = p * (dp - (p * dp).sum(-1, keepdim=True)) / D ** 0.5
    for got, w, x in ((o, p, f[2]), (dx, p.transpose(2, 3), f[3]), (dq, ds, f[1]), (dk, ds.transpose(2, 3), f[0])):
        ref = (w[..., None] * x[:, :, None]).sum(-2)
        err = (got.view(dims[0], 2, H, D).transpose(1, 2) - ref).abs().max().item()
        assert err <= 8 * TOL["f32"], err                      # sums of a few products up to 40


@pytest.mark.parametrize("n,D,tabled,window,valid", [(16, 64, False, 0, 0), (3, 36, True, 0, 100), (11, 64, False, 4, 0), (7, 100, True, 0, 0), (16, 128, False, 0, 333), (5, 128, False, 2, 0)])
def test_large_and_small_calls_give_the_same_bits(n, D, tabled, window, valid):
    """On 16-row tiles calls of more than 4,096 waves work visibility out at another place than smaller ones."""
    B, H, tiles = 16, 8, 40
    dims = (tiles * (16 // n) - (1 if n < 16 else 0), n)   # (the last tile is not full)
    assert B * H * tiles > 4096 > H * tiles
    gen = torch.Generator(device="cuda").manual_seed(8300 + n + D)
    q, k, v = (torch.randn((B, dims[0] * n, H, D), generator=gen, device="cuda") for _ in range(3))
    seen = torch.rand((n, n), generator=gen, device="cuda") < 0.7
    table = torch.from_numpy(ta.pack_axis_mask(seen.cpu().numpy())).cuda() if tabled else None

    def hop(q, k, v):
        plan = ta.ta_plan_create(q.shape[0], H, H, D, dims, ta.TA_F32, not tabled, window=(0, window), valid_len=valid, axis_masks=[None, table])
        o = torch.full_like(q, float("nan"))
        ta.ta_axis_attn_forward(plan, 1, q, k, v, ta.TA_VIN_O, o)
        return o
    whole = hop(q, k, v)
    assert torch.isfinite(whole).all()
    for b in (0, B - 1):
        assert torch.equal(whole[b:b + 1], hop(*(t[b:b + 1].contiguous() for t in (q, k, v))))
