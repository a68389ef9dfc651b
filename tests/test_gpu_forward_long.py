"""GPU parity of the long-axis forward at its edges: one and two key blocks that stay, the first axis that streams, rows one before
and after a block, a tile and a workgroup of four and of eight tiles, grouped and single heads, narrow rows, every mask, the encoding,
and scores that grow along the keys, so that the softmax's reference value moves with every tile."""
import numpy as np
import pytest
import torch

import paper_2410_20926_amd as ta
from gpu_util import TOL, multihop_forward
from oracle import tensattn_oracle as orc
from paper_2410_20926_amd.workloads import make_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # dims, B, Hq, Hkv, D, causal, window, valid_lens, rope base
    ((65, 2), 1, 2, 2, 128, True, None, None, None),
    ((3, 96), 2, 4, 2, 64, False, None, (288, 100), None),
    ((2, 127), 1, 4, 1, 128, True, None, None, None),
    ((128, 3), 1, 3, 1, 100, True, (40, 0), None, 10000.0),
    ((129, 2), 1, 2, 1, 128, False, None, None, None),
    ((192, 2), 1, 3, 3, 36, True, None, (301,), None),
    ((2, 257), 1, 2, 2, 64, True, (0, 70), None, 200.0),
    ((511,), 1, 2, 1, 128, True, None, None, None),
    ((513,), 2, 2, 2, 96, False, None, (513, 0), None),
    ((769, 2), 1, 4, 1, 128, True, (300, 0), None, None),
    ((1100,), 1, 2, 1, 64, True, None, None, 10000.0),
    ((200, 2), 1, 8, 2, 100, True, None, (390,), 10000.0),
    ((1030,), 2, 8, 2, 64, True, None, (1030, 500), None),      # four heads per workgroup
    ((1060,), 1, 4, 1, 100, False, (600,), None, 10000.0),      # the same, narrow rows
    ((1056, 8), 1, 64, 8, 40, True, None, (8000,), None),       # the same, more workgroups than CUs: two tiles of each head
    ((3, 90), 1, 8, 2, 128, True, None, (200,), 10000.0),       # later hop, heads that share K
    ((2, 70), 2, 4, 1, 64, False, (0, 40), None, None),
]


def forward_function(dims, axis, Hq, Hkv, D):
    """Four heads that share K side by side on up to four tiles, or below 1,024 positions (512 in 64-wide tiles) where they share the values too."""
    n = dims[axis]
    if Hq // Hkv % 4 == 0 and (n < (1024 if D > 64 else 512) if axis == 0 else n <= 96 and D in (64, 128)):
        return "mfma_fwd_stream_chunked_kernel" if n <= 128 else "mfma_fwd_stream_shared_kernel"
    return "mfma_fwd_long_kernel"


@pytest.mark.parametrize("dims,B,Hq,Hkv,D,causal,window,lens,rope", CASES)
def test_long_axis_forward_matches_oracle(dims, B, Hq, Hkv, D, causal, window, lens, rope):
    N = int(np.prod(dims))
    q, k, v = make_inputs(B, N, Hq, Hkv, D, seed=8500 + N + D, dtype="bf16")
    kw = dict(window=window, rope_base=rope)
    pkw = dict(kw)
    if lens is not None:
        pkw["valid_lens"] = torch.tensor(lens, dtype=torch.int64, device="cuda")
    got, plan, _ = multihop_forward(q, k, v, dims, "bf16", causal, **pkw)
    axis = int(np.argmax(dims))
    assert plan.hop_function(axis, ta.TA_VIN_KV if axis == 0 else ta.TA_VIN_O) == forward_function(dims, axis, Hq, Hkv, D)
    ref = orc.tensorized_attention_forward(q, k, v, dims, causal, valid_len=list(lens) if lens else None, **kw)
    err = np.abs(got - ref).max()
    assert np.isfinite(got).all() and err <= TOL["bf16"], f"{err:.3e}"


@pytest.mark.parametrize("n,growth", [(128, 0.02), (400, 0.02), (400, 0.3), (700, -0.3)])
def test_growing_scores_move_the_reference(n, growth):
    """Key c's score is growth * c times the query's size: the maximum of a row moves with every tile, by little and by much."""
    H, D = 2, 64
    q, k, v = make_inputs(1, n, H, H, D, seed=86, dtype="bf16")
    q[..., 0] = 8.0
    k[..., 0] = (growth * np.arange(n, dtype=np.float32)).astype(np.float32)[None, :, None]
    k = torch.from_numpy(k).to(torch.bfloat16).float().numpy()
    for causal in (False, True):
        got, _, _ = multihop_forward(q, k, v, (n,), "bf16", causal)
        ref = orc.tensorized_attention_forward(q, k, v, (n,), causal)
        err = np.abs(got - ref).max()
        assert np.isfinite(got).all() and err <= TOL["bf16"], f"causal={causal}: {err:.3e}"


@pytest.mark.parametrize("n,H,Hkv,D,causal,window,valid", [
    (100, 2, 2, 64, True, 0, 64), (128, 2, 2, 128, False, 0, 37), (128, 2, 1, 128, True, 0, 128), (200, 4, 1, 128, True, 0, 150),
    (300, 2, 2, 100, False, 40, 129), (1030, 4, 1, 64, True, 0, 700), (321, 2, 2, 128, True, 0, 321)])
def test_values_out_of_reach_stay_out(n, H, Hkv, D, causal, window, valid):
    """Keys are visible 32 at a time: an infinity or NaN in a value row that none of a query tile's 32 rows may see, nor any of the 31
    keys beside it, leaves the tile's output what it is without it (same bits); key tiles of padding reach no row, and padded
    rows give zeros."""
    q, k, v = (torch.from_numpy(x).cuda().to(torch.bfloat16) for x in make_inputs(1, n, H, Hkv, D, seed=871, dtype="bf16"))
    plan = ta.ta_plan_create(1, H, Hkv, D, (n,), ta.TA_BF16, causal, window=(window,), valid_len=valid)

    def run(k, v):
        o = torch.full_like(q, 7.0)
        ta.ta_axis_attn_forward(plan, 0, q, k, v, ta.TA_VIN_KV, o)
        return o.cpu()

    clean = run(k, v)
    assert (clean[:, valid:] == 0).all()
    bad_k, bad_v = k.clone(), v.clone()
    pad = (valid + 31) // 32 * 32
    bad_k[:, valid:], bad_v[:, pad:] = float("nan"), float("inf")
    bad_v[:, pad::2] = float("nan")
    if H // Hkv != 4 or n >= 1024:                         # (four heads that share K and the values, below 1,024: whole padded axes are walked)
        assert torch.equal(run(bad_k, bad_v), clean)
    for c in {min(45, valid - 1), (valid - 1) // 2, valid - 1}:
        bad_v = v.clone()
        bad_v[:, c] = float("inf")
        got = run(k, bad_v)
        for a0 in range(0, valid, 32):                     # query tiles none of whose rows sees any key of c's tile
            c0, a1 = c // 32 * 32, a0 + 31
            if (causal and c0 > a1) or (window and (c0 - a1 >= window or a0 - (c0 + 31) >= window)):
                assert torch.equal(got[:, a0:a1 + 1], clean[:, a0:a1 + 1]), (c, a0)
        assert not torch.isfinite(got[0, c]).any()


@pytest.mark.parametrize("n,D,causal", [(128, 64, False), (544, 128, False), (1088, 64, True), (2080, 128, False)])
def test_rounding_of_the_weights(n, D, causal):
    """Weights are rounded to bf16 relative to the row's largest score so far, 32 keys at a time, so that the largest weight is exact;
    the error against 64 bits is that of the same arithmetic in numpy (a reference that lags behind the maximum: 2 to 7 per cent more)."""
    H = 4
    q, k, v = make_inputs(1, n, H, H, D, seed=873 + n, dtype="bf16")
    got, _, _ = multihop_forward(q, k, v, (n,), "bf16", causal)
    bf16 = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16).double().numpy()
    Q, K, V = (bf16(x)[0].swapaxes(0, 1) for x in (q, k, v))
    s = Q @ K.swapaxes(1, 2) / np.sqrt(D)
    if causal:
        s = np.where(np.tril(np.ones((n, n), bool)), s, -np.inf)
    w = np.exp(s - s.max(-1, keepdims=True))
    exact = w @ V / w.sum(-1, keepdims=True)
    top, acc, l = np.full((H, n, 1), -np.inf), 0.0, 0.0
    for c in range(0, n, 32):
        now = np.maximum(top, s[:, :, c:c + 32].max(-1, keepdims=True))
        fade = np.exp(top - now)
        w = bf16(np.exp(s[:, :, c:c + 32] - now))
        acc, l, top = acc * fade + w @ V[:, c:c + 32], l * fade + w.sum(-1, keepdims=True), now
    want = bf16(acc / l)
    err, bound = (np.linalg.norm(x - exact) for x in (got[0].swapaxes(0, 1), want))
    assert err <= 1.005 * bound, f"{err / np.linalg.norm(exact):.4e}, with the exact reference {bound / np.linalg.norm(exact):.4e}"
