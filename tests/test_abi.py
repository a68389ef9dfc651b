"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header
declares, and its host logic (plan, cost model, error paths) behaves as documented.
No kernel is launched here."""
import ctypes as C
import json
import os
import re

import numpy as np
import pytest

import paper_2410_20926_amd as ta
from paper_2410_20926_amd import tensattn as binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "tensattn.h")
GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "paper_facts.json")


def declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ta_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = ta.load_library()
    names = declared_symbols()
    assert len(names) >= 21
    for name in names:
        assert hasattr(lib, name), f"{name} declared in tensattn.h but not exported"
    assert sorted(binding.EXPORTS) == names


def test_version_and_status_strings():
    assert ta.ta_version() == (0, 7)
    lib = ta.load_library()
    assert lib.ta_status_string(0) == b"TA_OK"
    assert lib.ta_status_string(5) == b"TA_ERR_ALIAS"


def test_plan_reshape_convention_matches_paper():
    fact = json.load(open(GOLDEN))["extrapolation_first_axis"]
    p = ta.ta_plan_create(1, 32, 8, 128, fact["dims"], ta.TA_BF16, True)
    assert p.seq_len() == fact["seq_len"]
    assert p.axis_stride(0) == fact["first_axis_increment_tokens"]
    assert [p.axis_stride(i) for i in range(3)] == [1024, 32, 1]
    assert [p.axis_fibres(i) for i in range(3)] == [1024, 1024, 1024]
    assert [p.hop_axis(i) for i in range(3)] == [0, 1, 2]          # Algorithm 1's order
    p = ta.ta_plan_create(1, 32, 8, 128, (64, 64, 32), ta.TA_BF16, True)
    assert [p.axis_stride(i) for i in range(3)] == [2048, 32, 1]
    assert [p.axis_fibres(i) for i in range(3)] == [2048, 2048, 4096]
    p = ta.ta_plan_create(1, 2, 2, 64, (4, 3), ta.TA_F32, False, hop_order=(1, 0))
    assert [p.hop_axis(i) for i in range(2)] == [1, 0]
    assert p.axis_stride(5) == -1 and p.hop_axis(2) == -1 and p.hop_kernel(0, 7) is None


def test_cost_model_closed_forms():
    B, Hq, Hkv, D, dims = 1, 32, 8, 128, (32, 32, 32)
    N = 32768
    p = ta.ta_plan_create(B, Hq, Hkv, D, dims, ta.TA_BF16, True)
    assert p.hop_bytes(0, ta.TA_VIN_KV) == B * N * D * 2 * (Hq + Hkv + Hkv + Hq) == 671088640
    assert p.hop_bytes(1, ta.TA_VIN_O) == B * N * D * 2 * (Hq + Hkv + Hq + Hq) == 872415232
    assert p.hop_bytes(0, ta.TA_VIN_KV) / N == 20480 and p.hop_bytes(1, ta.TA_VIN_O) / N == 26624
    for ax in range(3):
        assert p.hop_flops(ax) == 4.0 * B * Hq * N * dims[ax] * D
        assert p.hop_flops(ax, True) == 2.5 * p.hop_flops(ax)
    # backward: first processed hop (axis 2, value input = an O) overwrites dQ, dK
    assert p.hop_bytes(2, ta.TA_VIN_O, True, False) / N == 2 * D * (Hq + Hkv + Hq + Hq + Hq + Hq + Hkv) == 45056
    assert p.hop_bytes(1, ta.TA_VIN_O, True, True) / N == 55296
    assert p.hop_bytes(0, ta.TA_VIN_KV, True, True) / N == 43008
    o_bytes = B * N * Hq * D * 2
    # 32 x 32 x 32 in bf16 at D = 128: the last two hops run fused in inference, so one intermediate O
    assert p.fused_position() == 1 and p.pair_kernel(1, ta.TA_VIN_O) == "mfma_bf16_pair_n32"
    assert p.pair_bytes(1, ta.TA_VIN_O) / N == 26624
    assert p.workspace_bytes(False) == o_bytes and p.workspace_bytes(True) == 2 * o_bytes
    pw = ta.ta_plan_create(B, Hq, Hkv, D, (32, 16, 64), ta.TA_BF16, True)
    assert pw.fused_position() == -1 and pw.pair_kernel(1, ta.TA_VIN_O) == "unsupported"
    assert pw.workspace_bytes(False) == 2 * o_bytes
    assert p.backward_scratch_bytes() == 2 * o_bytes
    p1 = ta.ta_plan_create(1, 1, 1, 64, (256,), ta.TA_F32, False)
    assert p1.workspace_bytes(False) == 0
    p2 = ta.ta_plan_create(1, 1, 1, 64, (16, 16), ta.TA_F32, False)
    assert p2.workspace_bytes(False) == 256 * 64 * 4 and p2.workspace_bytes(True) == 256 * 64 * 4


@pytest.mark.parametrize("kw,status", [
    (dict(dims=()), "TA_ERR_SHAPE"),
    (dict(dims=(2,) * 9), "TA_ERR_SHAPE"),
    (dict(dims=(4, 0)), "TA_ERR_SHAPE"),
    (dict(dims=(4, -3)), "TA_ERR_SHAPE"),
    (dict(n_q_heads=6, n_kv_heads=4), "TA_ERR_SHAPE"),
    (dict(batch=0), "TA_ERR_SHAPE"),
    (dict(head_dim=101), "TA_ERR_UNSUPPORTED"),
    (dict(head_dim=512), "TA_ERR_UNSUPPORTED"),
    (dict(dtype=7), "TA_ERR_INVALID_ARG"),
    (dict(hop_order=(0, 0)), "TA_ERR_INVALID_ARG"),
    (dict(hop_order=(0, 2)), "TA_ERR_INVALID_ARG"),
    (dict(scale=-1.0), "TA_ERR_INVALID_ARG"),
    (dict(scale=float("nan")), "TA_ERR_INVALID_ARG"),
    (dict(q_strides=(64, 64, 64)), "TA_ERR_SHAPE"),             # overlapping rows
    (dict(o_strides=(4 * 3 * 2 * 64, 2 * 64, 60)), "TA_ERR_SHAPE"),   # not a multiple of 8
    (dict(dims=(1 << 20, 1 << 20, 1 << 20)), "TA_ERR_SHAPE"),   # overflow
    (dict(window=(0, -2)), "TA_ERR_INVALID_ARG"),
    (dict(valid_len=-1), "TA_ERR_INVALID_ARG"),
    (dict(valid_len=13), "TA_ERR_SHAPE"),
    (dict(valid_lens=0x1004), "TA_ERR_INVALID_ARG"),            # not 8-byte aligned
    (dict(rope_base=-2.0), "TA_ERR_INVALID_ARG"),
    (dict(rope_base=float("inf")), "TA_ERR_INVALID_ARG"),
])
def test_plan_rejects_bad_descriptors(kw, status):
    args = dict(batch=1, n_q_heads=2, n_kv_heads=2, head_dim=64, dims=(4, 3), dtype=ta.TA_F32, causal=False)
    args.update(kw)
    with pytest.raises(ta.TaError) as ei:
        ta.ta_plan_create(**args)
    assert ei.value.name == status
    assert ei.value.detail


def test_per_fibre_mask_flag_must_be_0_or_1_and_packing_keeps_the_fibre_axis():
    import numpy as np
    d = binding.make_desc(1, 2, 2, 64, (4, 3), ta.TA_F32, False)
    d.axis_mask_per_fibre[1] = 3
    with pytest.raises(ta.TaError) as e:
        ta.Plan(d)
    assert e.value.name == "TA_ERR_INVALID_ARG"
    d.axis_mask_per_fibre[1] = 1
    d.axis_mask_per_fibre[5] = 9                       # entries at or beyond `order` are ignored
    ta.Plan(d)
    m = np.random.default_rng(3).random((7, 40, 40)) < 0.5
    packed = ta.pack_axis_mask(m).view(np.uint32)
    assert packed.shape == (7, 40, 2)
    for f, a, c in ((0, 0, 0), (6, 39, 39), (3, 17, 32), (2, 5, 31)):
        assert bool((packed[f, a, c // 32] >> (c % 32)) & 1) == bool(m[f, a, c])
    assert np.array_equal(ta.pack_axis_mask(m[4]), ta.pack_axis_mask(m)[4])


def test_rope_flag_must_be_0_or_1():
    d = binding.make_desc(1, 2, 2, 64, (4, 3), ta.TA_F32, False)
    d.rope = 2
    with pytest.raises(ta.TaError) as e:
        ta.Plan(d)
    assert e.value.name == "TA_ERR_INVALID_ARG"
    # the encoding rides on the same kernels, the fused pair of hops included
    p = ta.ta_plan_create(1, 32, 8, 128, (32, 32, 32), ta.TA_BF16, True, rope_base=10000.0)
    assert p.fused_position() == 1 and p.pair_kernel(1, ta.TA_VIN_O) == "mfma_bf16_pair_n32"
    assert p.workspace_bytes(False) == 32768 * 32 * 128 * 2
    assert p.hop_kernel(1, ta.TA_VIN_O) == "mfma_bf16_n32_shared" and p.hop_backward_kernel(1, ta.TA_VIN_O) == "mfma_bf16_bwd_n32"


def test_plan_create_null_pointers():
    lib = ta.load_library()
    h = C.c_void_p()
    assert lib.ta_plan_create(None, C.byref(h)) == 1
    d = binding.make_desc(1, 1, 1, 64, (4,), ta.TA_F32, False)
    assert lib.ta_plan_create(C.byref(d), None) == 1
    lib.ta_plan_destroy(None)
    assert lib.ta_plan_seq_len(None) == -1
    assert lib.ta_plan_workspace_bytes(None, 0) == 0


def test_strided_layouts_accepted():
    # head-major [B, H, N, D] for every tensor
    B, H, N, D = 2, 4, 12, 64
    s = (H * N * D, D, N * D)
    p = ta.ta_plan_create(B, H, H, D, (3, 4), ta.TA_BF16, True, q_strides=s, kv_strides=s, o_strides=s)
    assert p.seq_len() == 12


def test_strides_whose_span_would_overflow_are_refused():
    """A stride so large that (extent - 1) * stride leaves the 64-bit range is a shape error, not an
    address wrap in the alias checks."""
    huge = (1 << 60, 64, 8 * 64)
    with pytest.raises(ta.TaError) as ei:
        ta.ta_plan_create(16, 8, 8, 64, (4, 4), ta.TA_BF16, True, q_strides=huge)
    assert ei.value.name == "TA_ERR_SHAPE"
    ok = (1 << 40, 8 * 64, 64)
    assert ta.ta_plan_create(16, 8, 8, 64, (4, 4), ta.TA_BF16, True, q_strides=ok).seq_len() == 16


def test_entry_points_reject_bad_arguments_without_launching():
    """All of these return before any HIP call, so they run without a GPU.  The
    addresses are fabricated and never dereferenced."""
    p = ta.ta_plan_create(1, 2, 1, 64, (4, 3), ta.TA_F32, True)
    nbytes_q = 12 * 2 * 64 * 4
    Q, K, V, O, W = 0x10000000, 0x20000000, 0x30000000, 0x40000000, 0x50000000

    def status(fn, *a, **k):
        with pytest.raises(ta.TaError) as ei:
            fn(*a, **k)
        return ei.value.name

    S = 0xdead0   # never used: the calls fail first
    assert status(ta.ta_axis_attn_forward, p, 2, Q, K, V, 0, O, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_axis_attn_forward, p, -1, Q, K, V, 0, O, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_axis_attn_forward, p, 0, Q, K, V, 3, O, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_axis_attn_forward, p, 0, None, K, V, 0, O, S) == "TA_ERR_NULL"
    assert status(ta.ta_axis_attn_forward, p, 0, Q, K, V, 0, None, S) == "TA_ERR_NULL"
    assert status(ta.ta_axis_attn_forward, p, 0, Q + 4, K, V, 0, O, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_axis_attn_forward, p, 0, Q, K, V, 0, Q + nbytes_q - 16, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_axis_attn_forward, p, 0, Q, K, V, 0, V, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_axis_attn_forward, p, 0, Q, K, O, 1, O, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_forward, p, Q, K, V, O, None, 0, False, S) == "TA_ERR_NULL"
    assert status(ta.ta_multihop_forward, p, Q, K, V, O, W, 16, False, S) == "TA_ERR_WORKSPACE"
    assert status(ta.ta_multihop_forward, p, Q, K, V, O, W + 16, 1 << 20, False, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_multihop_forward, p, Q, K, V, O, O, 1 << 20, False, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_forward, p, None, K, V, O, W, 1 << 20, False, S) == "TA_ERR_NULL"
    assert status(ta.ta_axis_attn_backward, p, 0, Q, K, V, 0, O, Q, W, W + (1 << 20), False, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_axis_attn_backward, p, 0, Q, K, V, 0, O, W, W, W + (1 << 20), False, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_axis_attn_backward, p, 0, Q, K, V, 0, None, W, W, W, False, S) == "TA_ERR_NULL"
    assert status(ta.ta_multihop_backward, p, Q, K, V, O, W, 16, W, W, W, W, 0, S) == "TA_ERR_WORKSPACE"
    assert status(ta.ta_rope_apply, p, 2, 0, Q, O, 0.0, False, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_rope_apply, p, 0, 2, Q, O, 0.0, False, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_rope_apply, p, 0, -1, Q, Q + 32, 0.0, False, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_rope_apply, p, 0, -1, None, O, 0.0, False, S) == "TA_ERR_NULL"
    assert status(ta.ta_rope_apply, p, 1, 0, Q, O, -3.0, False, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_copy_bytes, Q, K, 24, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_copy_bytes, None, K, 32, S) == "TA_ERR_NULL"
    assert status(ta.ta_stream_mix, Q, K, 4, 5, 3, S) == "TA_ERR_UNSUPPORTED"      # no kernel for that mix
    assert status(ta.ta_stream_mix, None, K, 4, 1, 1, S) == "TA_ERR_NULL"
    assert status(ta.ta_stream_mix, Q + 8, K, 4, 1, 1, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_stream_slabs, Q, K, V, None, 1024, 4, 2, 1, S) == "TA_ERR_NULL"
    assert status(ta.ta_stream_slabs, Q, K, V, O, 1000, 4, 2, 1, S) == "TA_ERR_INVALID_ARG"   # not a multiple of 1024
    assert status(ta.ta_stream_slabs, Q, K, V, O, 1024, 4, 3, 1, S) == "TA_ERR_INVALID_ARG"   # heads do not divide
    assert status(ta.ta_stream_slabs, Q, K, V, O, 1024, 4, 2, 4, S) == "TA_ERR_INVALID_ARG"   # no such granule
    assert status(ta.ta_stream_slabs, Q, K, V, O + 8, 1024, 4, 2, 1, S) == "TA_ERR_INVALID_ARG"


def test_multihop_calls_validate_every_hop_before_the_first_launch():
    """Nothing may be enqueued when a call is going to fail: aliasing, alignment and the
    availability of a kernel for EVERY hop are checked up front.  There is no GPU here, so a
    call that got as far as a launch would come back as TA_ERR_DEVICE instead."""
    def status(fn, *a, **k):
        with pytest.raises(ta.TaError) as ei:
            fn(*a, **k)
        return ei.value.name

    S = 0xdead0
    Q, K, V, O, W, G = 0x10000000, 0x20000000, 0x30000000, 0x40000000, 0x50000000, 0x60000000
    DQ, DK, DV, SC = 0x70000000, 0x80000000, 0x90000000, 0xa0000000
    p = ta.ta_plan_create(1, 2, 1, 64, (4, 3), ta.TA_F32, True)
    big = 1 << 20
    # the output of the LAST hop overlaps an input: found before the first hop is enqueued
    assert status(ta.ta_multihop_forward, p, Q, K, V, Q + 64, W, big, False, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_forward, p, Q, K, V, V, W, big, False, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_forward, p, Q, K + 8, V, O, W, big, False, S) == "TA_ERR_INVALID_ARG"
    # backward: scratch and workspace are range-checked against every tensor and each other
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, DQ, DK, DV, W, big, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, DQ, DK, DV, DQ, big, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, DQ, DK, DV, Q, big, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, W, DK, DV, SC, big, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, DQ, DQ, DV, SC, big, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, DQ, DK, K, SC, big, S) == "TA_ERR_ALIAS"
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, DQ, DK, DV, SC + 16, big, S) == "TA_ERR_INVALID_ARG"
    assert status(ta.ta_multihop_backward, p, Q, K, V, G, W, big, DQ + 2, DK, DV, SC, big, S) == "TA_ERR_INVALID_ARG"
    # an fp32 axis too long for the backward's row statistics: the hop over axis 1 runs first in
    # the backward and is fine, the hop over axis 0 is not; the call must refuse before either
    long_axis = ta.ta_plan_create(1, 8, 1, 64, (4096, 2), ta.TA_F32, True)
    assert long_axis.hop_backward_kernel(1, ta.TA_VIN_O) == "generic"
    assert long_axis.hop_backward_kernel(0, ta.TA_VIN_KV) == "unsupported"
    huge = 1 << 28
    A = [i << 32 for i in range(1, 12)]
    assert status(ta.ta_multihop_backward, long_axis, A[0], A[1], A[2], A[3], A[4], huge, A[5], A[6], A[7], A[8], huge, S) == "TA_ERR_UNSUPPORTED"


def test_launch_geometry_is_settled_when_the_plan_is_made():
    """Whether a kernel's launch grid fits is decided by ta_plan_create, not at launch time."""
    ok = ta.ta_plan_create(32767, 1, 1, 64, (32769, 16), ta.TA_BF16, True)
    assert ok.hop_kernel(1, ta.TA_VIN_KV) == "mfma_bf16_n32" and ok.hop_backward_kernel(1, ta.TA_VIN_KV) == "mfma_bf16_bwd_n32"
    # 32,769 tiles need 2 grid rows per batch element: with 32,768 batch elements no grid holds the job, neither
    # the matrix-core kernel's nor the generic kernel's, and the plan says so (it used to surface as a failed launch)
    more = ta.ta_plan_create(32768, 1, 1, 64, (32769, 32), ta.TA_BF16, True)
    assert more.hop_kernel(1, ta.TA_VIN_KV) == "unsupported"
    assert more.hop_backward_kernel(1, ta.TA_VIN_KV) == "generic"        # one workgroup per fibre and group: that grid fits
    assert more.pair_kernel(0, ta.TA_VIN_KV) == "unsupported"
    none = ta.ta_plan_create(65535, 8, 1, 64, (32769, 32), ta.TA_BF16, True)         # more workgroups than any grid here holds
    assert none.hop_kernel(1, ta.TA_VIN_KV) == "unsupported"
    with pytest.raises(ta.TaError) as e:
        ta.ta_axis_attn_forward(none, 1, 1 << 50, 2 << 50, 3 << 50, ta.TA_VIN_KV, 4 << 50, 0xdead0)
    assert e.value.name == "TA_ERR_UNSUPPORTED"


def test_sequence_length_overflow_is_caught_before_multiplying():
    for dims in ((1 << 30, 1 << 30), (1 << 20, 1 << 20, 1 << 20), (2147483647, 2147483647, 2147483647, 2147483647)):
        with pytest.raises(ta.TaError) as e:
            ta.ta_plan_create(1, 1, 1, 64, dims, ta.TA_F32, False)
        assert e.value.name == "TA_ERR_SHAPE"
    assert ta.load_library().ta_status_string(8) == b"TA_ERR_NOMEM"


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", "/nonexistent/libtensattn.so")
    with pytest.raises(ImportError):
        ta.ta_plan_create(1, 1, 1, 64, (4,), ta.TA_F32, False)


def test_pack_axis_mask_layout():
    """Row a, word c // 32, bit c % 32 (the layout the descriptor's axis_mask documents)."""
    rng = np.random.default_rng(5)
    for n in (1, 5, 32, 33, 70):
        m = rng.random((n, n)) < 0.5
        words = ta.pack_axis_mask(m).view(np.uint32)
        assert words.shape == (n, (n + 31) // 32)
        for a in range(n):
            for c in range(n):
                assert ((int(words[a, c // 32]) >> (c % 32)) & 1) == int(m[a, c])
        # bits past the last column are zero
        if n % 32:
            assert (words[:, -1] >> np.uint32(n % 32) == 0).all()


def test_misaligned_axis_mask_is_rejected():
    with pytest.raises(ta.TaError) as e:
        ta.Plan(binding.make_desc(1, 2, 2, 64, (4, 4), ta.TA_F32, True, axis_masks=[6, None]))
    assert e.value.name == "TA_ERR_INVALID_ARG"


def test_kernels_for_other_head_widths():
    p = ta.ta_plan_create(1, 32, 32, 100, (32, 32), ta.TA_BF16, True)      # OpenLLaMA-3B geometry: a multiple of 4
    assert p.hop_kernel(0, ta.TA_VIN_KV) == "mfma_bf16_n32" and p.hop_kernel(1, ta.TA_VIN_O) == "mfma_bf16_n32"
    # the fused kernel takes the width, but the multi-hop call uses it only for rows of whole 64-byte pieces (widths
    # that are a multiple of 32): elsewhere the two hops on their own are faster
    assert p.fused_position() == -1 and p.pair_kernel(0, ta.TA_VIN_KV) == "mfma_bf16_pair_n32"
    assert ta.ta_plan_create(1, 32, 8, 96, (32, 32), ta.TA_BF16, True).fused_position() == 0
    assert p.hop_backward_kernel(1, ta.TA_VIN_O) == "mfma_bf16_bwd_n32"
    two_tiles = ta.ta_plan_create(1, 32, 32, 100, (64, 16), ta.TA_BF16, True)
    assert two_tiles.hop_kernel(0, ta.TA_VIN_KV) == "mfma_bf16_n64"
    assert two_tiles.hop_backward_kernel(0, ta.TA_VIN_KV) == "mfma_bf16_bwd_blocked"      # narrow heads: no two-tile form
    assert ta.ta_plan_create(1, 32, 8, 128, (64, 16), ta.TA_BF16, True).hop_backward_kernel(0, ta.TA_VIN_KV) == "mfma_bf16_bwd_n64"
    long_axis = ta.ta_plan_create(1, 8, 2, 96, (128, 4), ta.TA_BF16, True)
    assert long_axis.hop_kernel(0, ta.TA_VIN_KV) == "mfma_bf16_stream_shared_kv"
    odd = ta.ta_plan_create(1, 4, 4, 90, (16, 16), ta.TA_BF16, True)       # even, not a multiple of 4
    assert odd.hop_kernel(0, ta.TA_VIN_KV) == "generic"


def test_device_functions_of_a_plan():
    """ta_plan_hop_function tells apart what shares one plan name, and ta_plan_small_pair_position says where two hops are one launch."""
    def fn(Hq, Hkv, D, dims, axis, vin, backward, dtype=ta.TA_BF16):
        return ta.ta_plan_create(1, Hq, Hkv, D, dims, dtype, True).hop_function(axis, vin, backward)
    KV, O = ta.TA_VIN_KV, ta.TA_VIN_O
    assert fn(4, 4, 64, (16, 4), 0, KV, False, ta.TA_F32) == "f32_fwd_kernel" and fn(4, 4, 64, (33, 4), 0, KV, False, ta.TA_F32) == "f32_fwd_long_kernel"
    assert fn(4, 4, 64, (32, 4), 0, KV, True, ta.TA_F32) == "f32_bwd_kernel" and fn(4, 4, 64, (33, 4), 0, KV, True, ta.TA_F32) == "f32_bwd_long_kernel"
    assert fn(4, 4, 90, (16, 4), 0, KV, False, ta.TA_F32) == "generic_forward_kernel" and fn(4, 4, 130, (16, 4), 0, KV, True) == "generic_backward_kernel"
    assert fn(8, 2, 128, (32, 4), 0, KV, False) == "mfma_fwd_shared_kernel" and fn(8, 8, 128, (64, 4), 0, KV, False) == "mfma_fwd_kernel"
    assert fn(8, 2, 128, (128, 4), 0, KV, False) == "mfma_fwd_stream_chunked_kernel" and fn(8, 2, 128, (129, 4), 0, KV, False) == "mfma_fwd_stream_shared_kernel"
    assert fn(8, 2, 128, (96, 4), 0, O, False) == "mfma_fwd_stream_chunked_kernel" and fn(8, 2, 128, (97, 4), 0, O, False) == "mfma_fwd_long_kernel"
    assert fn(8, 2, 100, (96, 4), 0, O, False) == "mfma_fwd_long_kernel" and fn(8, 2, 128, (1024, 4), 0, KV, False) == "mfma_fwd_long_kernel"
    assert fn(8, 8, 128, (200, 4), 0, KV, False) == "mfma_fwd_long_kernel"
    assert fn(8, 2, 128, (32, 4), 0, KV, True) == "mfma_bwd_kernel" and fn(8, 2, 128, (40, 4), 0, KV, True) == "mfma_bwd2_kernel"
    assert fn(8, 2, 128, (40, 256), 0, KV, True) == "mfma_bwd_resident_kernel" and fn(24, 4, 128, (64, 4), 0, KV, True) == "mfma_bwd_resident_kernel"
    assert fn(8, 2, 128, (130, 4), 0, KV, True) == "mfma_bwd_long_kernel" and fn(8, 2, 128, (130, 128), 0, KV, True) == "mfma_bwd_stream_kernel"
    assert fn(8, 1, 64, (4096, 2), 0, KV, True, ta.TA_F32) == "unsupported" and fn(8, 2, 128, (16, 4), 2, KV, False) is None
    small = lambda *a, **k: ta.ta_plan_create(1, *a, ta.TA_BF16, True, **k).small_pair_position()
    assert small(8, 2, 128, (5, 10, 9)) == 1 and small(8, 2, 128, (10, 9)) == 0
    assert small(8, 2, 128, (32, 16, 16)) == 1 and small(4, 4, 128, (3, 16, 16)) == -1       # two tiles per wave: from 256 slabs of a head on
    assert small(8, 2, 100, (5, 10, 9)) == -1 and small(8, 2, 128, (32, 32)) == -1 and small(8, 2, 128, (10, 9), hop_order=(1, 0)) == -1


def test_traffic_of_several_instantiations_is_averaged():
    from paper_2410_20926_amd import counters
    rec = counters.traffic_record({
        "mfma_bwd_resident_kernel<128, 2, 1, false, false>": {"FETCH_SIZE": 4.0, "WRITE_SIZE": 2.0, "launches": 1},
        "mfma_bwd_resident_kernel<128, 2, 2, false, false>": {"FETCH_SIZE": 1.0, "WRITE_SIZE": 1.0, "launches": 3},
        "mfma_fwd_shared_kernel<128, 1, true, false, false>": {"FETCH_SIZE": 5.0, "WRITE_SIZE": 3.0, "launches": 7}})
    assert rec == {"mfma_bwd_resident_kernel": {"fetch_bytes_per_launch": 1.75, "write_bytes_per_launch": 1.25},
                   "mfma_bf16_n32_shared_kv": {"fetch_bytes_per_launch": 5.0, "write_bytes_per_launch": 3.0}}


def test_kernel_names_with_enumerators():
    """A profiler writes an enumerator among a kernel's template arguments with its type."""
    from paper_2410_20926_amd.counters import short
    ns, end = "void ta::(anonymous namespace)::", "(ta::BwdParams, ta::mfma::TileParams)"
    assert short(ns + "mfma_bwd_kernel<128, false, false, (ta::(anonymous namespace)::BwdRows)1, false>" + end) == "mfma_bwd_kernel<128, false, false, 1, false>"
    assert short(ns + "mfma_fwd_long_kernel<64, 8, (ta::(anonymous namespace)::Form)2, true, false>(ta::HopParams)") == "mfma_fwd_long_kernel<64, 8, 2, true, false>"
    assert short(ns + "copy_kernel(void*)") == "copy_kernel" and short("void at::native::sum_kernel<1>(int)") is None


def test_forms_of_the_long_axis_forward():
    """Windows that are short against a workgroup and bit tables are not run in phases; axes of 1,024 to 2,047 positions are where the workgroups come out even."""
    FOUR, EIGHT, PHASES = "four_tiles_in_step", "eight_tiles_in_step", "eight_tiles_in_phases"

    def form(n, B, Hq, Hkv, D, causal=True, window=0, table=False, rope=None, vin=ta.TA_VIN_KV, lens=None):
        # (a table's address, and that of lengths, is only kept here)
        return ta.ta_plan_create(B, Hq, Hkv, D, (n,), ta.TA_BF16, causal, window=(window,), axis_masks=[0x1000 if table else None], rope_base=rope, valid_lens=lens).hop_form(0, vin)
    assert form(128, 8, 8, 8, 128) == "two_blocks" and form(200, 8, 8, 8, 128) == FOUR
    for Hq, Hkv, D, least in ((32, 8, 128, 1280), (8, 8, 128, 1536), (32, 8, 64, 2048), (16, 16, 64, 2048)):
        assert form(4096, 4, Hq, Hkv, D) == PHASES and form(2048, 8, Hq, Hkv, D) == PHASES
        for w in (64, 256, least - 1):
            assert form(4096, 4, Hq, Hkv, D, window=w) == FOUR
        assert form(4096, 4, Hq, Hkv, D, window=least) == PHASES
        assert form(4096, 4, Hq, Hkv, D, False, window=least // 2) == FOUR and form(4096, 4, Hq, Hkv, D, False, window=least // 2 + 1) == PHASES
        assert form(4096, 4, Hq, Hkv, D, table=True) == FOUR and form(1500, 8, Hq, Hkv, D, table=True) == FOUR
        assert form(4096, 4, Hq, Hkv, D, rope=0.0) == EIGHT
    for Hq, Hkv, D, least in ((12, 12, 100, 3000), (16, 4, 100, 3000), (8, 8, 40, 1024)):
        assert form(4096, 8, Hq, Hkv, D) == PHASES and form(4095, 8, Hq, Hkv, D) == EIGHT
        assert form(4096, 8, Hq, Hkv, D, window=least - 1) == EIGHT and form(4096, 8, Hq, Hkv, D, window=least) == PHASES
        assert form(4096, 8, Hq, Hkv, D, table=True) == EIGHT
    assert form(1023, 8, 12, 12, 100) == FOUR
    assert form(4096, 1, 1, 1, 128) == FOUR                # 16 workgroups of eight tiles for 256 CUs
    # 1,024 to 2,047 positions
    assert form(2047, 4, 8, 8, 128, False) == PHASES and form(2047, 4, 8, 8, 128) == PHASES and form(2047, 4, 8, 8, 64) == PHASES     # 256 workgroups
    assert form(2047, 4, 8, 8, 128, lens=0x1000) == FOUR and form(2048, 4, 8, 8, 128, lens=0x1000) == PHASES
    assert form(1500, 8, 8, 8, 128, False) == FOUR         # 384: the second round half empty
    assert form(1024, 8, 32, 8, 128) == FOUR and form(1024, 8, 32, 8, 128, False) == PHASES      # equal waves under the mask as it is
    assert form(2047, 4, 8, 8, 128, False, window=2046) == PHASES and form(2047, 4, 8, 8, 128, False, window=300) == FOUR
    assert ta.ta_plan_create(1, 8, 2, 128, (16, 16), ta.TA_BF16, True).hop_form(0, ta.TA_VIN_KV) == "" and ta.ta_plan_create(1, 8, 2, 128, (16, 16), ta.TA_BF16, True).hop_form(2, 0) is None


def test_forms_of_the_one_tile_backward():
    """Narrow rows: pairs of heads where workgroups of one are not dealt out in order and there are waves for the chip, streamed where the call is a little
    larger than the last-level cache; whole rows have one form."""
    CACHED, STREAMED, PAIRS = "rows_cached", "rows_streamed", "heads_in_pairs"

    def form(n, fibres, B, Hq, Hkv, D, vin=ta.TA_VIN_KV, rope=None):
        return ta.ta_plan_create(B, Hq, Hkv, D, (n, fibres), ta.TA_BF16, True, rope_base=rope).hop_form(0, vin, True)

    def streamed(Hq, Hkv, D, vin):                         # fibres of 32 rows from and up to which a call streams
        rows = [form(32, 8 * i, 1, Hq, Hkv, D, vin) for i in range(1, 700)]
        first = rows.index(STREAMED)
        assert set(rows[:first]) == {CACHED} and set(rows[first:]) <= {CACHED, STREAMED, PAIRS}
        mb = 32 * 8 * D * 2 * (3 * Hq + 2 * Hkv + 2 * (Hq if vin else Hkv)) / 1e6
        return (first + 1) * mb, (first + 1 + rows[first:].index(CACHED)) * mb, mb
    for Hq, Hkv, D, vin, end in ((8, 8, 100, 1, 560), (8, 8, 40, 0, 450), (16, 4, 96, 0, 1400), (16, 4, 112, 1, 1400), (32, 2, 40, 1, 450)):
        low, high, step = streamed(Hq, Hkv, D, vin)
        assert 280 <= low < 280 + step and end <= high < end + step
    assert form(32, 123, 4, 12, 12, 100) == PAIRS and form(32, 124, 4, 12, 12, 100) == CACHED      # 1,476 and 1,488 workgroups of one head
    assert form(16, 246, 4, 12, 12, 40) == PAIRS and form(32, 60, 4, 11, 11, 100) == CACHED and form(32, 61, 4, 24, 12, 100) == CACHED
    assert form(32, 53, 2, 12, 12, 100) == CACHED and form(32, 55, 2, 12, 12, 100) == PAIRS         # 1,272 and 1,320 waves
    assert form(32, 303, 4, 12, 12, 100) == PAIRS          # (651 MB and out of order)
    # large calls whose pairs are in order too: 32 heads of 32 x 32 x 32, 1.47 GB; 0.73 GB of width 100, 112, 96 (whole sectors) and 112 on packed tiles
    assert form(32, 1024, 1, 32, 32, 100) == PAIRS and form(32, 512, 1, 32, 32, 100) == CACHED and form(32, 512, 1, 32, 32, 112) == PAIRS
    assert form(32, 1024, 1, 32, 32, 96) == CACHED and form(16, 1024, 1, 32, 32, 112) == CACHED and form(32, 3001, 1, 8, 8, 100) == CACHED
    assert form(32, 1024, 1, 32, 32, 100, rope=0.0) == CACHED and form(32, 1024, 1, 32, 32, 112, rope=0.0) == form(32, 123, 4, 12, 12, 100, rope=0.0) == PAIRS
    assert form(32, 123, 4, 12, 12, 128) == "" and form(33, 123, 4, 12, 12, 100) == ""


def test_forms_of_the_long_backward():
    """Few fibres go in parts, a call that fills the chip does not."""
    def form(n, fibres, Hq, Hkv, D, B=1, causal=True, vin=ta.TA_VIN_KV, **kw):
        plan = ta.ta_plan_create(B, Hq, Hkv, D, (n, fibres), ta.TA_BF16, causal, **kw)
        assert plan.hop_function(0, vin, True) == "mfma_bwd_long_kernel"
        return plan.hop_form(0, vin, True)
    for vin in (ta.TA_VIN_KV, ta.TA_VIN_O):
        assert form(1024, 8, 8, 8, 128, vin=vin) == "in_parts" and form(1024, 16, 8, 8, 128, vin=vin) == form(256, 256, 8, 8, 128, vin=vin) == "whole"
        assert form(300, 40, 8, 2, 64, vin=vin) == "in_parts" and form(300, 80, 8, 2, 64, vin=vin) == form(300, 10, 8, 2, 64, B=8, vin=vin) == "whole"
        assert form(129, 1, 1, 1, 40, causal=False, vin=vin) == "in_parts"
        # the calls whose bits are compared in test_gpu_backward_parts.py: a batch, and one of its elements
        for n, fibres, B, Hq, Hkv, D, causal, kw in ((129, 9, 32, 4, 2, 64, True, {}), (256, 8, 32, 3, 3, 128, True, {}), (257, 8, 32, 2, 2, 40, False, dict(rope_base=500.0)),
                                                     (300, 6, 40, 4, 2, 100, True, dict(window=(40, 0))), (520, 2, 130, 4, 2, 64, True, dict(rope_base=1e4)),
                                                     (330, 3, 96, 6, 2, 128, False, dict(window=(100, 0)))):
            assert form(n, fibres, Hq, Hkv, D, B, causal, vin, **kw) == "whole" and form(n, fibres, Hq, Hkv, D, 1, causal, vin, **kw) == "in_parts"


def test_forms_of_the_one_and_two_tile_forward():
    """Rows of up to 60 features: through the caches, but streamed on two tiles in calls a little larger than the last-level cache; wider narrow rows: streamed."""
    def form(n, fibres, Hq, Hkv, D, vin=ta.TA_VIN_KV):
        return ta.ta_plan_create(1, Hq, Hkv, D, (n, fibres), ta.TA_BF16, True).hop_form(0, vin)
    for Hq, Hkv, D, vin in ((8, 8, 40, 0), (8, 2, 40, 1), (6, 2, 20, 1)):
        mb = 50 * D * 2 * (2 * Hq + Hkv + (Hq if vin else Hkv)) / 1e6
        for at, streamed in ((270, False), (281, False), (283, True), (389, True), (391, False), (1000, False)):
            assert form(50, round(at / mb), Hq, Hkv, D, vin) == ("rows_streamed" if streamed else "rows_cached")
            assert form(25, round(2 * at / mb), Hq, Hkv, D, vin) == "rows_cached"
    assert {form(50, i, 8, 2, 40, 0) for i in range(200, 8000, 200)} == {"rows_cached"}      # a group's heads share the values
    assert form(50, 10, 8, 2, 100) == form(20, 10, 8, 8, 72) == "rows_streamed" and form(50, 10, 8, 2, 128) == form(20, 10, 8, 8, 64) == ""


def test_forms_of_the_wide_narrow_forward():
    """Rows of 65 to 127 features: streamed below 16 MB and from 282 to 480 MB, through the caches elsewhere, on either number of tiles, grouped or not."""
    def form(n, fibres, Hq, Hkv, D, vin, **kw):
        return ta.ta_plan_create(1, Hq, Hkv, D, (n, fibres), ta.TA_BF16, True, **kw).hop_form(0, vin)
    for n, Hq, Hkv, D, vin in ((50, 8, 2, 100, 0), (20, 8, 8, 72, 1), (32, 16, 4, 96, 1), (33, 3, 3, 124, 0)):
        mb = n * D * 2 * (2 * Hq + Hkv + (Hq if vin else Hkv)) / 1e6
        for at, streamed in ((1, True), (15, True), (17, False), (281, False), (283, True), (479, True), (481, False), (1000, False)):
            for kw in ({}, dict(rope_base=1e4)):
                assert form(n, round(at / mb), Hq, Hkv, D, vin, **kw) == ("rows_streamed" if streamed else "rows_cached")


def test_stream_lookup_without_torch_private_names(monkeypatch):
    """A torch that has dropped the private way to the current stream's handle is asked for a stream object."""
    import torch
    asked = []
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: asked.append(1) or type("S", (), {"cuda_stream": 77}))
    for gone in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        with monkeypatch.context() as m:
            m.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 55 + device, raising=False)
            m.setattr(torch._C, "_cuda_getDevice", lambda: 1, raising=False)
            assert binding._stream(None) == 56 and not asked
            m.delattr(torch._C, gone)
            assert binding._stream(None) == 77 and asked.pop()
