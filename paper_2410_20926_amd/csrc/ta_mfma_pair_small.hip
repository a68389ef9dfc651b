// The last two hops of Algorithm 1 in one launch for small slabs (the two innermost axes hold at most 256 tokens, each axis at most 32
// positions), bf16, gfx950: the hop along the second-innermost axis, then the hop along the innermost one (Eq. 4 twice with the
// same Q and K).  The value tensor between them stays in LDS.
//
// A workgroup is one slab (n1 x n2 consecutive tokens) of one head.  Both hops are cut into 32-row tiles of whole fibres, as in the
// one-tile kernel: column tiles (fibres along n1, rows n2 tokens apart) for the first, row tiles (consecutive tokens) for the
// second; a wave has kTiles of each.  It gathers Q, K and the value rows of its column tiles and Q and K of its row tiles
// (the second read of a row finds it in L2), forms both softmaxes and the column tiles' P1 X; when every wave has its own, the
// results go to LDS, and after a barrier the row tiles take them from there as value operand.  Against two launches a
// head's Q and K cross HBM once instead of twice, and the tensor between the hops not at all.  What bounds it: the memory's rate for 256-byte
// rows at an 8 KB pitch (a head per workgroup; the one-tile kernels take four heads of a token together), and two dependent
// rounds of gathers per wave above 128 tokens.  32 x 16 x 16 tokens, 32 heads of width 128, all three hops: 143 -> 126 us;
// 500 x 15 x 16, 8 heads of width 64: 441 -> 323 us; 8 x 10 x 10, 8 heads: 20.6 -> 15.6 us.
#include "ta_mfma_common.h"

namespace ta {
namespace {

using namespace mfma;
template <bool NARROW, int N>
__device__ inline void ready_rows(u32x4 (&raw)[N], uint32_t mis, const char*, uint32_t, uint32_t lbyte, uint32_t dbytes) {
    if constexpr (NARROW) {
#pragma unroll
        for (int i = 0; i < N; ++i) raw[i] = gather_ready<NARROW>(raw[i], (mis >> i) & 1u, lbyte, dbytes);
    }
}


constexpr int kWaves = 4;
constexpr int kMaxSlab = 256;

struct SmallParams {
    uint32_t slabs, units;                                // slabs per batch element; B * slabs * Hq
    int32_t fpt1, t1, fpt2, t2;                           // fibres per tile and tiles of a slab, column tiles and row tiles
    uint32_t q_row, k_row, v_row, o_row;                  // token pitch in bytes
    void* mid;                                            // nullptr, or an O-shaped tensor for the first hop's output
};

// NARROW: the head is narrower than the D-wide tile; see gather_request.
template <int D, int kTiles, bool NARROW, bool ROPE>
__global__ __launch_bounds__(64 * kWaves, 2) void mfma_fwd_pair_small_kernel(HopParams h1, HopParams h2, SmallParams sp) {
    using G = Geo<D>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t u = blockIdx.y * gridDim.x + blockIdx.x;     // head fastest
    if (u >= sp.units) return;                            // whole workgroup leaves together
    const int h = (int)(u % (uint32_t)h1.Hq);
    u /= (uint32_t)h1.Hq;
    const uint32_t slab = u % sp.slabs;
    const int b = (int)(u / sp.slabs);
    const int g = h / h1.G, hv = h1.vin_heads == h1.Hq ? h : g;
    const int n1 = h1.n, n2 = h2.n;
    const uint32_t tok0 = slab * (uint32_t)(n1 * n2);
    const char* qb = reinterpret_cast<const char*>(h1.q.p) + ((int64_t)b * h1.q.sb + (int64_t)h * h1.q.sh) * 2;
    const char* kb = reinterpret_cast<const char*>(h1.k.p) + ((int64_t)b * h1.k.sb + (int64_t)g * h1.k.sh) * 2;
    const char* xb = reinterpret_cast<const char*>(h1.vin.p) + ((int64_t)b * h1.vin.sb + (int64_t)hv * h1.vin.sh) * 2;
    const int64_t oslice = ((int64_t)b * h1.o.sb + (int64_t)h * h1.o.sh) * 2;
    char* ob = reinterpret_cast<char*>(h1.o.p) + oslice;
    char* mb = reinterpret_cast<char*>(sp.mid) + oslice;

    const int lrow = lane / G::kChunks, lcol = lane % G::kChunks;
    const uint32_t lbyte = lcol * 16;
    const uint32_t dbytes = (uint32_t)h1.D * 2;
    const int r32 = lane & 31, hf = lane >> 5;
    float rev[4];
    if constexpr (ROPE) rope_rates(h1, lcol, rev);
    const int64_t vl = hop_valid_len(h1, b);

    // slab row of tile row r of column tile t (fibres t * fpt1 ..) / row tile t, and how many rows the tile has
    auto rows1 = [&](int t) { return min(sp.fpt1, n2 - t * sp.fpt1) * n1; };
    auto rows2 = [&](int t) { return min(sp.fpt2, n1 - t * sp.fpt2) * n2; };
    auto row1 = [&](int t, int r) { const int fl = r / n1; return (r - fl * n1) * n2 + t * sp.fpt1 + fl; };
    auto row2 = [&](int t, int r) { return t * sp.fpt2 * n2 + r; };

    char* buf = smem + w * (kTile * G::kPitch);           // this wave's transit tile until the first barrier
    char* stg = buf + lrow * G::kPitch + lbyte;
    const char* nat = buf + r32 * G::kPitch + hf * 16;

    u32x4 p2[kTiles][2], mid[kTiles][G::kDTiles * 2];     // row tiles' weights; column tiles' results, rounded
    float inv2[kTiles];
    // weights of a tile (un-normalised, maximum 1, rounded) and 1 / their sum
    auto softmax = [&](const f32x16& st, uint32_t vis, u32x4 (&pop)[2]) {
        const float sl2 = h1.scale * kLog2e;
        float m = -INFINITY, l = 0.f, corr;
        online_softmax_tile(st, vis, hf, sl2, m, l, pop, corr);
        return l > 0.f ? 1.f / l : 0.f;
    };
    // keys (tile rows) that this lane's row of a tile sees: fibre number fl of the tile, position a of an axis of n, first token of the fibre
    auto visible = [&](const HopParams& p, int fl, int a, int count, uint32_t first, int64_t fibre) {
        if (fl >= count) return 0u;
        const int64_t left = vl - (int64_t)first;
        const int nreal = left <= 0 ? 0 : (int)min((int64_t)p.n, (left + p.stride - 1) / p.stride);
        if (a >= nreal) return 0u;
        int lo, hi;
        visible_range(a, 0, p.n, p.causal, p.window, lo, hi);
        uint32_t v = range_mask(lo, min(hi, nreal));
        if (p.mask) v &= table_word(p, (uint32_t)fibre, a, 0);
        return v << (fl * p.n);
    };

#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
        const int t = w + i * kWaves;
        if (t >= sp.t1 && t >= sp.t2) continue;
        __builtin_amdgcn_sched_barrier(0);
        u32x4 q1[G::kPasses], k1[G::kPasses], x1[G::kPasses], q2[G::kPasses], k2[G::kPasses];
        const int c1 = rows1(min(t, sp.t1 - 1)), c2 = rows2(min(t, sp.t2 - 1));   // a wave with a tile of one kind only works on the other kind's last one too and keeps nothing of it
        const int ta = min(t, sp.t1 - 1), tb = min(t, sp.t2 - 1);
        uint32_t mq1 = 0u, mk1 = 0u, mx1 = 0u, mq2 = 0u, mk2 = 0u;   // NARROW: a bit per request, see gather_request
#pragma unroll
        for (int j = 0; j < G::kPasses; ++j) {
            const uint32_t tok = tok0 + (uint32_t)row1(ta, min(j * G::kRowsPerPass + lrow, c1 - 1));
            q1[j] = gather_noted<NARROW, false>(qb, tok * sp.q_row, lbyte, dbytes, j, mq1);
            k1[j] = gather_noted<NARROW, false>(kb, tok * sp.k_row, lbyte, dbytes, j, mk1);
            x1[j] = gather_noted<NARROW, false>(xb, tok * sp.v_row, lbyte, dbytes, j, mx1);
        }
#pragma unroll
        for (int j = 0; j < G::kPasses; ++j) {
            const uint32_t tok = tok0 + (uint32_t)row2(tb, min(j * G::kRowsPerPass + lrow, c2 - 1));
            q2[j] = gather_noted<NARROW, false>(qb, tok * sp.q_row, lbyte, dbytes, j, mq2);
            k2[j] = gather_noted<NARROW, false>(kb, tok * sp.k_row, lbyte, dbytes, j, mk2);
        }
        __builtin_amdgcn_sched_barrier(0);
        auto scores = [&](u32x4 (&q)[G::kPasses], u32x4 (&k)[G::kPasses], uint32_t mq, uint32_t mk, int n, int count) {
            ready_rows<NARROW>(q, mq, qb, sp.q_row, lbyte, dbytes);
            ready_rows<NARROW>(k, mk, kb, sp.k_row, lbyte, dbytes);
            if constexpr (ROPE) {
#pragma unroll
                for (int j = 0; j < G::kPasses; ++j) {
                    const float pos = (float)(min(j * G::kRowsPerPass + lrow, count - 1) % n);
                    q[j] = rope_chunk(q[j], pos, rev);
                    k[j] = rope_chunk(k[j], pos, rev);
                }
            }
            u32x4 qop[G::kKSteps];
            lds_wave_sync();
            stage_rows<D>(stg, q);
            lds_wave_sync();
            read_natural<D>(nat, qop);
            lds_wave_sync();
            stage_rows<D>(stg, k);
            lds_wave_sync();
            f32x16 st = {};
#pragma unroll
            for (int s = 0; s < G::kKSteps; ++s) st = mma(*reinterpret_cast<const u32x4*>(nat + 32 * s), qop[s], st);
            return st;
        };
        // column tile: scores, weights, P1 X
        u32x4 pop[2];
        const int fa = r32 / n1, aa = r32 - fa * n1;
        const f32x16 s1 = scores(q1, k1, mq1, mk1, n1, c1);
        const float inv1 = softmax(s1, visible(h1, fa, aa, c1 / n1, tok0 + (uint32_t)(ta * sp.fpt1 + fa), (int64_t)slab * n2 + ta * sp.fpt1 + fa), pop);
        ready_rows<NARROW>(x1, mx1, xb, sp.v_row, lbyte, dbytes);
        lds_wave_sync();
        stage_rows<D>(stg, x1);
        lds_wave_sync();
        u32x4 xT[G::kDTiles][2];
        read_transposed<D>(buf + (4 * hf + ((lane & 15) >> 2)) * G::kPitch + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2, xT);
#pragma unroll
        for (int d = 0; d < G::kDTiles; ++d) {
            f32x16 o = {};
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) o = mma(xT[d][s2], pop[s2], o);
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
                mid[i][2 * d + s2] = u32x4{pack_bf16x2(o[8 * s2] * inv1, o[8 * s2 + 1] * inv1), pack_bf16x2(o[8 * s2 + 2] * inv1, o[8 * s2 + 3] * inv1),
                                           pack_bf16x2(o[8 * s2 + 4] * inv1, o[8 * s2 + 5] * inv1), pack_bf16x2(o[8 * s2 + 6] * inv1, o[8 * s2 + 7] * inv1)};
        }
        // row tile: scores, weights
        const int fb = r32 / n2, ab = r32 - fb * n2;
        const f32x16 s2t = scores(q2, k2, mq2, mk2, n2, c2);
        inv2[i] = softmax(s2t, visible(h2, fb, ab, c2 / n2, tok0 + (uint32_t)((tb * sp.fpt2 + fb) * n2), (int64_t)slab * n1 + tb * sp.fpt2 + fb), p2[i]);
    }
    __syncthreads();                                      // the transit tiles are done with: the slab takes their place
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
        const int t = w + i * kWaves;
        if (t < sp.t1 && r32 < rows1(t)) {
            char* row = smem + row1(t, r32) * G::kPitch;
#pragma unroll
            for (int d = 0; d < G::kDTiles; ++d)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    const u32x4 v = mid[i][2 * d + s2];
                    *reinterpret_cast<u32x2*>(row + (32 * d + 16 * s2 + 4 * hf) * 2) = u32x2{v.x, v.y};
                    *reinterpret_cast<u32x2*>(row + (32 * d + 16 * s2 + 8 + 4 * hf) * 2) = u32x2{v.z, v.w};
                }
        }
    }
    __syncthreads();                                      // the slab is complete
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
        const int t = w + i * kWaves;
        if (t >= sp.t2) continue;
        const int count = rows2(t);                       // the tile's rows belong to this wave alone from here on
        char* base = smem + row2(t, 0) * G::kPitch;
        auto store = [&](char* out) {
#pragma unroll
            for (int j = 0; j < G::kPasses; ++j) {
                const int r = j * G::kRowsPerPass + lrow;
                if (r < count)
                    store_row_chunk<NARROW, G::kChunks>(out, (tok0 + (uint32_t)row2(t, r)) * sp.o_row, base + r * G::kPitch + lbyte, lbyte, dbytes);
            }
        };
        if (sp.mid) store(mb);
        f32x16 o[G::kDTiles];
        // transposed value operand; rows past the tile read its last row (their weights are zero)
        const int tr = 4 * hf + ((lane & 15) >> 2), tc = (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
#pragma unroll
        for (int d = 0; d < G::kDTiles; ++d) {
            o[d] = f32x16{};
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const char* a0 = base + min(16 * s2 + tr, count - 1) * G::kPitch + tc + 64 * d;
                const char* a1 = base + min(16 * s2 + 8 + tr, count - 1) * G::kPitch + tc + 64 * d;
                const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0)));
                const u32x2 y = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a1)));
                o[d] = mma(u32x4{x.x, x.y, y.x, y.y}, p2[i][s2], o[d]);
            }
        }
        lds_wave_sync();
        if (r32 < count) {
#pragma unroll
            for (int d = 0; d < G::kDTiles; ++d)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    u32x2 v;
                    v.x = pack_bf16x2(o[d][4 * q4] * inv2[i], o[d][4 * q4 + 1] * inv2[i]);
                    v.y = pack_bf16x2(o[d][4 * q4 + 2] * inv2[i], o[d][4 * q4 + 3] * inv2[i]);
                    *reinterpret_cast<u32x2*>(base + r32 * G::kPitch + (32 * d + 8 * q4 + 4 * hf) * 2) = v;
                }
        }
        lds_wave_sync();
        store(ob);
    }
}

template <int D, int kTiles, bool NARROW, bool ROPE>
hipError_t launch(const HopParams& h1, const HopParams& h2, const SmallParams& sp, hipStream_t s) {
    const int rows = h1.n * h2.n > kWaves * kTile ? h1.n * h2.n : kWaves * kTile;
    const int smem = rows * Geo<D>::kPitch;
    if (smem > 64 * 1024) {
        const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(mfma_fwd_pair_small_kernel<D, kTiles, NARROW, ROPE>), smem);
        if (e != hipSuccess) return e;
    }
    const uint32_t x = sp.units < 1048576u ? sp.units : 1048576u;
    hipLaunchKernelGGL((mfma_fwd_pair_small_kernel<D, kTiles, NARROW, ROPE>), dim3(x, (sp.units + x - 1) / x), dim3(64 * kWaves), smem, s, h1, h2, sp);
    return hipGetLastError();
}
template <int D, bool NARROW>
hipError_t launch(const HopParams& h1, const HopParams& h2, const SmallParams& sp, hipStream_t s) {
    const bool two = sp.t1 > kWaves || sp.t2 > kWaves;
    if (h1.rope) return two ? launch<D, 2, NARROW, true>(h1, h2, sp, s) : launch<D, 1, NARROW, true>(h1, h2, sp, s);
    return two ? launch<D, 2, NARROW, false>(h1, h2, sp, s) : launch<D, 1, NARROW, false>(h1, h2, sp, s);
}

// False where the slab does not fit or two launches are faster.
bool small_params(const HopParams& h1, const HopParams& h2, SmallParams* sp) {
    if (h1.n < 1 || h2.n < 1 || h1.n > kTile || h2.n > kTile || h1.n * h2.n > kMaxSlab || h2.stride != 1 || h1.stride != h2.n) return false;
    if (h1.D < 8 || h1.D > 128 || h1.D % 4 != 0 || !mfma_forward_layout_ok(h1)) return false;
    sp->fpt1 = kTile / h1.n; sp->t1 = (h2.n + sp->fpt1 - 1) / sp->fpt1;
    sp->fpt2 = kTile / h2.n; sp->t2 = (h1.n + sp->fpt2 - 1) / sp->fpt2;
    if (sp->t1 > 2 * kWaves || sp->t2 > 2 * kWaves) return false;
    // Fewer than three tiles leave most waves idle (four sequences of 200 x 4 x 5, 16 / 4 heads: 199 against the two launches' 121 us; 64 x 8 x 8, two
    // tiles: level), and rows narrower than 128 in 128-wide tiles do not leave registers for five tiles in flight (100 x 12 x 12, 32 heads of
    // width 100: 369 against 356 us).
    if (sp->t1 < 3 && sp->t2 < 3) return false;
    if (h1.D > 64 && h1.D < 128) return false;
    const int64_t slabs = h1.fibres * h1.n / (h1.n * h2.n), units = slabs * h1.B * h1.Hq;
    if (units <= 0 || units > 0x7fffffffLL) return false;
    // Two tiles per wave are two rounds of gathers one after the other: on fewer slabs than CUs the two launches are done sooner (one head of
    // 9 x 12 x 15: 24.3 against 17.5 us; 8 sequences of 16 x 16, 32 heads, 256 slabs: 22.4 against 27.8).
    if ((sp->t1 > kWaves || sp->t2 > kWaves) && units < 256) return false;
    sp->slabs = (uint32_t)slabs;
    sp->units = (uint32_t)units;
    sp->q_row = (uint32_t)(h1.q.st * 2); sp->k_row = (uint32_t)(h1.k.st * 2);
    sp->v_row = (uint32_t)(h1.vin.st * 2); sp->o_row = (uint32_t)(h1.o.st * 2);
    return true;
}

}  // namespace

bool mfma_pair_small_supports(const HopParams& h1, const HopParams& h2, int dtype) {
    SmallParams sp;
    return dtype == TA_BF16 && small_params(h1, h2, &sp);
}

hipError_t launch_mfma_forward_pair_small(const HopParams& h1, const HopParams& h2, void* o_mid, hipStream_t s) {
    SmallParams sp;
    if (!small_params(h1, h2, &sp)) return hipErrorInvalidValue;
    sp.mid = o_mid;
    return h1.D == 128 ? launch<128, false>(h1, h2, sp, s) : h1.D == 64 ? launch<64, false>(h1, h2, sp, s) : launch<64, true>(h1, h2, sp, s);
}

}  // namespace ta
