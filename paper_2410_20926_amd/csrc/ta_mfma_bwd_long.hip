// bf16 MFMA backward for axes of more than four tiles (128 < n <= 1024), gfx950.  The derivative itself is that of
// ta_mfma_bwd.hip.
//
// A workgroup of eight waves is one fibre of one key/value head (up to eight query heads of its group per launch), because
// the row statistics of the fibre have to be at hand for every key tile and live in LDS.  Eight 32-row tiles are worked
// on at a time, a wave each, its own rows held as operands, and the rows of the other side stream past all of them in blocks
// of 64, once into LDS for eight tiles (two buffers, one barrier per block, the block after next requested when a block is
// written):
//   query side, per head and eight query tiles:   K and the value input stream twice: S^T and dP^T for the row statistics
//                (running max, sum, sum of P o dP), then again for dS^T and dQ^T = K^T dS^T;
//   key side, per eight key tiles:   the heads' Q and dO stream once: S and dP with a key per lane, dX^T += dO^T P and
//                dK^T += Q^T dS, summed over the heads in registers.
// A call of few fibres, which would leave most of the chip idle, goes in parts: the query side of eight tiles of a head and the key side of eight tiles are
// workgroups of their own, the latter with the statistics once more (parts_of).
// What bounds it: the chain of one wave's step (two score products, softmax arithmetic, two contractions, twice per block), with two waves
// per SIMD; five tiles leave three waves idle.  The blocked kernel gathers a tile per wave and visit and waits for it.  Backward hops,
// width 128 causal: 8 heads of 1,024 x 16 2,790 -> 416 us, 32 / 8 heads of 256 x 128 1,150 -> 776 us, of 200 x 64 513 -> 386 us (along the first axis, a value input per head; 424 while what
// depends on the lane was kept in registers and the key side spilled 52); width 64: 8 heads
// of 512 x 64 622 -> 161 us.
#include "ta_mfma_bwd_common.h"
#include <algorithm>
#include <cmath>
#include <type_traits>

namespace ta {
namespace {

using namespace mfma;

constexpr int kWaves = 8;
constexpr int kRowsB = 64;                                // streamed rows of a block

template <int D>
struct LongGeo {
    static constexpr int kBlock = kRowsB * Geo<D>::kPitch;
    static constexpr int kStream = 4 * kBlock > kWaves * BGeo<D>::kBufBytes ? 4 * kBlock : kWaves * BGeo<D>::kBufBytes;   // two buffers of two tensors; also a transit tile per wave
    static constexpr int kFixed = kStream + kWaves * kTile * 16;
};

// NARROW: the head is narrower than the D-wide tile; see gather_request.  VS: the value input is per key/value head.  PARTS: a workgroup is a part of that (parts_of;
// instantiated on its own, since the bounds of a part cost the whole 2 to 4 per cent).
template <int D, bool VS, bool NARROW, bool ROPE, bool PARTS>
__global__ __launch_bounds__(64 * kWaves, 2) void mfma_bwd_long_kernel(BwdParams bp, StreamBwdParams sp) {
    using G = BGeo<D>;
    using L = LongGeo<D>;
    constexpr int kRowsPass = kWaves * G::kRowsPerPass;   // rows the workgroup fetches per pass
    constexpr int kMine = kRowsB / kRowsPass;
    // Narrow rows in 64-wide tiles, the value input shared: a third of the scalar registers that the loops spill belongs to row buffers and to the two ways of putting
    // rows together, so that a tile of its own is put together row by row and stored under a branch (32 / 8 heads of 40, 67 x 463 x 2, 1,550 -> 1,596 us with them, 1,527
    // now; of 60, 100 x 200 113 -> 116, now 111; per-head values and 128-wide tiles 1 to 3 per cent behind that way).
    constexpr bool kRowByRow = NARROW && VS && D == 64, kBranch = !NARROW || kRowByRow;
    const HopParams& p = bp.hop;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t bx, by;
    workgroup_xy<NARROW>(bx, by);
    const int g = (int)bx;
    const uint32_t zp = blockIdx.z / sp.fibres_hi;        // the longest parts of every fibre first
    const int part = PARTS ? (int)(zp / (uint32_t)p.B) : 0;
    const uint32_t zb = zp - (uint32_t)part * (uint32_t)p.B;
    const int64_t f = (int64_t)(blockIdx.z - zp * sp.fibres_hi) * sp.fibres_lo + by;
    if (f >= p.fibres) return;                            // whole workgroup leaves together
    const int b = (int)zb;
    const int n = p.n, T = sp.tiles;
    const uint32_t stride = (uint32_t)p.stride;
    const uint32_t tok0 = (uint32_t)fibre_base_token(f, p.stride, n);
    const uint32_t vl = (uint32_t)hop_valid_len(p, b);
    const int nreal = tok0 >= vl ? 0 : (int)min((uint32_t)n, (vl - tok0 + stride - 1) / stride);
    char* transit = smem + w * G::kBufBytes;
    u32x4* rowoff = reinterpret_cast<u32x4*>(smem + L::kStream) + w * kTile;
    float* stats = reinterpret_cast<float*>(smem + L::kFixed);   // [head][tile][max | 1 / sum | delta][32]

    const uint32_t dbytes = (uint32_t)p.D * 2;
    const float sl2 = p.scale * kLog2e;

    // What depends on the lane is formed again where it is used: kept over the loops below it would be spilled, and a reload waits for the
    // blocks requested before it.
    auto again = [](int x) {
        if (D == 128) asm volatile("" : "+v"(x));
        return x;
    };
    // But for the two products of a step where the heads of a group share the value input: whole rows have the registers there, and the arithmetic is in the chain (16 / 4
    // heads of 128, 1,000 x 40, 1,482 -> 1,535 us with it, 1,471 now; 8 / 2, 700 x 60, encoded, 938 -> 981, now 929; 32 / 8, 200 x 64, 328 -> 319, now 312).
    auto hot = [&](int x) { return VS && !NARROW ? x : again(x); };
    auto chunk_byte = [&]() { return (uint32_t)(again(lane) % G::kChunks) * 16u; };
    auto slice = [&](const Tensor& t, int head) { return reinterpret_cast<char*>(t.p) + ((int64_t)b * t.sb + (int64_t)head * t.sh) * 2; };
    // rows of tile t as operands contracted over the features, through this wave's transit tile
    auto own = [&](const char* base, uint32_t pitch, int t, bool turn, u32x4 (&op)[G::kKSteps]) {
        u32x4 raw[G::kPasses];
        uint32_t mis = 0u;
        const int lane_ = again(lane), lrow = lane_ / G::kChunks, r32 = lane_ & 31, hf = lane_ >> 5;
        const uint32_t lbyte = (uint32_t)(lane_ % G::kChunks) * 16u;
#pragma unroll
        for (int i = 0; i < G::kPasses; ++i) {
            raw[i] = gather_noted<NARROW, false>(base, (tok0 + (uint32_t)min(kTile * t + i * G::kRowsPerPass + lrow, n - 1) * stride) * pitch, lbyte, dbytes, i, mis);
            if constexpr (kRowByRow) raw[i] = gather_ready<NARROW>(raw[i], (mis >> i) & 1u, lbyte, dbytes);
        }
        if constexpr (!kRowByRow) gather_ready_all<NARROW>(raw, mis, base, pitch, lbyte, dbytes);
        if (ROPE && turn) {
            float rev[4];
            rope_rates(p, lane_ % G::kChunks, rev);
#pragma unroll
            for (int i = 0; i < G::kPasses; ++i) raw[i] = rope_chunk(raw[i], (float)min(kTile * t + i * G::kRowsPerPass + lrow, n - 1), rev);
        }
        lds_wave_sync();
        stage_rows<D>(transit + lrow * G::kPitch + lbyte, raw);
        lds_wave_sync();
        read_natural<D>(transit + r32 * G::kPitch + hf * 16, op);
    };
    auto set_rowoff = [&](int t) {
        lds_wave_sync();
        if (lane < kTile) {
            const uint32_t tok = tok0 + (uint32_t)min(kTile * t + lane, n - 1) * stride;
            rowoff[lane] = u32x4{tok * sp.q_row, tok * sp.k_row, tok * sp.v_row, tok * sp.o_row};
        }
        lds_wave_sync();
    };
    // Streams blocks [jb, je) of two tensors through LDS; work(j, first tensor's block, second tensor's block).  The first
    // tensor's rows are turned by their position when the hop encodes positions.  ahead() requests the first block and has to
    // come before; after a stream the first block is on its way again (for another sweep).  Nobody may be reading
    // the stream buffers when it is called, and nobody is when it returns.
    struct Raw { u32x4 v[kMine]; uint32_t mis; };
    struct Two { const char *base1, *base2; uint32_t pitch1, pitch2; int jb, je; };
    Raw ra, rc;
    auto request = [&](const char* base, uint32_t pitch, int j, Raw& raw) {
        const int myrow = w * G::kRowsPerPass + again(lane) / G::kChunks;
        const uint32_t lbyte = chunk_byte();
        raw.mis = 0u;
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const uint32_t r = (uint32_t)min(j * kRowsB + i * kRowsPass + myrow, n - 1);   // past the end: the last row, never visible
            uint32_t mis;
            raw.v[i] = gather_request<NARROW, false>(base, (tok0 + r * stride) * pitch, lbyte, dbytes, mis);
            raw.mis |= mis ? 1u << i : 0u;
        }
    };
    auto ahead = [&](const Two& t) {
        request(t.base1, t.pitch1, t.jb, ra);
        request(t.base2, t.pitch2, t.jb, rc);
    };
    auto stream = [&](const Two& t, auto work) {
        auto write = [&](char* block, int j, const Raw& raw, bool turn) {
            const int myrow = w * G::kRowsPerPass + again(lane) / G::kChunks;
            const uint32_t lbyte = chunk_byte();
            float rev[4];
            if (ROPE && turn) rope_rates(p, (int)lbyte / 16, rev);
#pragma unroll
            for (int i = 0; i < kMine; ++i) {
                u32x4 x = gather_ready<NARROW>(raw.v[i], (raw.mis >> i) & 1u, lbyte, dbytes);
                if (ROPE && turn) x = rope_chunk(x, (float)min(j * kRowsB + i * kRowsPass + myrow, n - 1), rev);
                *reinterpret_cast<u32x4*>(block + (i * kRowsPass + myrow) * G::kPitch + lbyte) = x;
            }
        };
        write(smem, t.jb, ra, true);
        write(smem + 2 * L::kBlock, t.jb, rc, false);
        int next = t.jb + 1 < t.je ? t.jb + 1 : t.jb;
        request(t.base1, t.pitch1, next, ra);
        request(t.base2, t.pitch2, next, rc);
        __syncthreads();
#pragma unroll 1
        for (int j = t.jb; j < t.je; ++j) {
            const int slot = (j - t.jb) & 1;
            if (j + 1 < t.je) {
                write(smem + (slot ^ 1) * L::kBlock, j + 1, ra, true);
                write(smem + (2 + (slot ^ 1)) * L::kBlock, j + 1, rc, false);
            }
            next = j + 2 < t.je ? j + 2 : t.jb;
            request(t.base1, t.pitch1, next, ra);
            request(t.base2, t.pitch2, next, rc);
            work(j, smem + slot * L::kBlock, smem + (2 + slot) * L::kBlock);
            __syncthreads();
        }
    };
    auto scores = [&](const char* tile, const u32x4 (&op)[G::kKSteps]) {
        f32x16 x = {};
        const int l = hot(lane);
        const char* at = tile + (l & 31) * G::kPitch + (l >> 5) * 16;
#pragma unroll
        for (int s = 0; s < G::kKSteps; ++s) x = mma(*reinterpret_cast<const u32x4*>(at + 32 * s), op[s], x);
        return x;
    };
    // scores that the lane's row (key) does not see become -inf; blocks that all of them see whole are left alone
    auto hide = [&](f32x16& st, uint32_t vis) {
        if (__all(vis == 0xffffffffu)) return;
        vis >>= 4 * (again(lane) >> 5);
#pragma unroll
        for (int r = 0; r < 16; ++r) st[r] = ((vis >> (8 * (r / 4) + (r % 4))) & 1u) ? st[r] : -INFINITY;
    };
    // acc^T += (tile)^T w, contracted over the tile's rows
    auto contract = [&](const char* tile, const u32x4 (&wt)[2], f32x16 (&acc)[G::kDTiles]) {
        const int l = hot(lane);
        const char* from = tile + (4 * (l >> 5) + ((l & 15) >> 2)) * G::kPitch + (16 * ((l >> 4) & 1) + 4 * (l & 3)) * 2;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int t = 0; t < G::kDTiles; ++t) {
                const char* a0 = from + 16 * s2 * G::kPitch + 64 * t;
                const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0)));
                const u32x2 y = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0 + 8 * G::kPitch)));
                acc[t] = mma(u32x4{x.x, x.y, y.x, y.y}, wt[s2], acc[t]);
            }
    };
    // rows [first, last] see keys of tiles [lo, hi); keys [first, last] are seen by rows of tiles [lo, hi)
    auto reach = [&](bool keys, int first, int last, int& lo, int& hi) {
        int l1, h1, l2, h2;
        first = min(first, n - 1); last = min(last, n - 1);
        if (keys) { seen_range(first, 0, n, p.causal, p.window, l1, h1); seen_range(last, 0, n, p.causal, p.window, l2, h2); }
        else { visible_range(first, 0, n, p.causal, p.window, l1, h1); visible_range(last, 0, n, p.causal, p.window, l2, h2); }
        lo = max(l1, 0) / kTile;
        hi = (min(h2, n) + kTile - 1) / kTile;
    };

    // This workgroup's share (parts_of): everything; or, first in the order of workgroups, the key side of eight tiles, which needs the statistics of the
    // rows that see them; or the query side of eight tiles of one head.  What a part forms it forms as the whole does.
    const int eights = (T + kWaves - 1) / kWaves;
    int h0 = 0, h1 = bp.wg_heads, a0b = 0, a0e = T, c0b = 0, c0e = T;
    const bool keys_only = PARTS && part < eights;
    if (keys_only) {
        int lo, hi;
        c0b = kWaves * part;
        c0e = min(T, c0b + kWaves);
        reach(true, kTile * c0b, kTile * c0e - 1, lo, hi);
        a0b = lo / kWaves * kWaves;
        a0e = hi;
    } else if (PARTS) {
        const int i = (part - eights) / bp.wg_heads;
        h0 = part - eights - i * bp.wg_heads;
        h1 = h0 + 1;
        a0b = kWaves * (eights - 1 - i);
        a0e = min(T, a0b + kWaves);
        c0e = 0;
    }

    // ===== query side ================================================================================
#pragma unroll 1
    for (int hl = h0; hl < h1; ++hl) {
        const int h = g * p.G + bp.head_base + hl;
        const char* xb = slice(p.vin, VS ? g : h);
        char* dqb = slice(bp.dq, h);
#pragma unroll 1
        for (int a0 = a0b; a0 < a0e; a0 += kWaves) {
            const int a = a0 + w;                         // past the last tile: the wave only fetches
            int lo, hi, wlo, whi;
            reach(false, kTile * a0, kTile * (a0 + kWaves) - 1, lo, hi);
            reach(false, kTile * a, kTile * a + kTile - 1, wlo, whi);
            if (a >= T) whi = wlo;
            const Two keys = {slice(p.k, g), xb, sp.k_row, sp.v_row, lo / 2, (hi + 1) / 2};
            ahead(keys);
            u32x4 qop[G::kKSteps], gop[G::kKSteps];
            own(slice(p.q, h), sp.q_row, min(a, T - 1), true, qop);
            own(slice(bp.d_o, h), sp.o_row, min(a, T - 1), false, gop);
            float m = -INFINITY, l = 0.f, dn = 0.f;
            __syncthreads();                              // the transit tiles are done with
            stream(keys, [&](int j, const char* kt, const char* xt) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int c = 2 * j + i;
                    if (c < wlo || c >= whi) continue;
                    f32x16 st = scores(kt + i * kTile * G::kPitch, qop);
                    const f32x16 dp = scores(xt + i * kTile * G::kPitch, gop);
                    hide(st, block_vis_keys(p, f, kTile * a + (again(lane) & 31), c, nreal));
                    float tmax = st[0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) tmax = fmaxf(tmax, st[r]);
                    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
                    const float mnew = fmaxf(m, tmax == -INFINITY ? tmax : tmax * sl2);
                    const float msafe = mnew == -INFINITY ? 0.f : mnew;
                    const float corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - msafe);
                    float ps = 0.f, pd = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float ev = __builtin_amdgcn_exp2f(fmaf(st[r], sl2, -msafe));
                        ps += ev;
                        pd += ev * dp[r];
                    }
                    l = l * corr + ps;                    // this lane's half of the row; joined below
                    dn = dn * corr + pd;
                    m = mnew;
                }
            });
            l += __shfl_xor(l, 32);
            dn += __shfl_xor(dn, 32);
            const float msafe = m == -INFINITY ? 0.f : m;
            const float inv = l > 0.f ? 1.f / l : 0.f;
            const float delta = dn * inv;
            if (lane < kTile && a < T) {
                float* sh = stats + (hl * T + a) * 3 * kTile;
                sh[lane] = msafe; sh[kTile + lane] = inv; sh[2 * kTile + lane] = delta;
            }
            if (keys_only) continue;
            f32x16 acc[G::kDTiles];
#pragma unroll
            for (int t = 0; t < G::kDTiles; ++t) acc[t] = f32x16{};
            stream(keys, [&](int j, const char* kt, const char* xt) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int c = 2 * j + i;
                    if (c < wlo || c >= whi) continue;
                    f32x16 st = scores(kt + i * kTile * G::kPitch, qop);
                    const f32x16 dp = scores(xt + i * kTile * G::kPitch, gop);
                    hide(st, block_vis_keys(p, f, kTile * a + (again(lane) & 31), c, nreal));
                    float ds[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r) ds[r] = __builtin_amdgcn_exp2f(fmaf(st[r], sl2, -msafe)) * (inv * (dp[r] - delta));
                    u32x4 wt[2];
                    pack_rows(ds, wt);
                    contract(kt + i * kTile * G::kPitch, wt, acc);
                }
            });
            if (a < T) {
                set_rowoff(a);
                u32x4 old[G::kDTiles * 2] = {};
                if (bp.accumulate) prefetch_tile<D, NARROW>(old, rowoff, 0, dqb, again(lane), dbytes);
                store_tile<D, NARROW, kBranch>(acc, p.scale, transit, rowoff, 0, dqb, old, bp.accumulate != 0, min(kTile, n - kTile * a), again(lane), dbytes,
                                      unrope(&p, [&](int r) { return (float)(kTile * a + r); }));
            }
        }
    }
    // ===== key side ==================================================================================
#pragma unroll 1
    for (int c0 = c0b; c0 < c0e; c0 += kWaves) {
        const int c = c0 + w;
        u32x4 kop[G::kKSteps], xop[G::kKSteps];
        own(slice(p.k, g), sp.k_row, min(c, T - 1), true, kop);
        if (VS) own(slice(p.vin, g), sp.v_row, min(c, T - 1), false, xop);
        int lo, hi, wlo, whi;
        reach(true, kTile * c0, kTile * (c0 + kWaves) - 1, lo, hi);
        reach(true, kTile * c, kTile * c + kTile - 1, wlo, whi);
        if (c >= T) whi = wlo;
        f32x16 dk[G::kDTiles], dx[G::kDTiles];
#pragma unroll
        for (int t = 0; t < G::kDTiles; ++t) { dk[t] = f32x16{}; dx[t] = f32x16{}; }
        const int rows_c = min(kTile, n - kTile * c);
#pragma unroll 1
        for (int hl = 0; hl < bp.wg_heads; ++hl) {
            const int h = g * p.G + bp.head_base + hl;
            const Two rows = {slice(p.q, h), slice(bp.d_o, h), sp.q_row, sp.o_row, lo / 2, (hi + 1) / 2};
            ahead(rows);
            if (!VS) {
                own(slice(p.vin, h), sp.v_row, min(c, T - 1), false, xop);
#pragma unroll
                for (int t = 0; t < G::kDTiles; ++t) dx[t] = f32x16{};
            }
            __syncthreads();                              // the transit tiles are done with, the statistics are there
            stream(rows, [&](int j, const char* qt, const char* gt) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int a = 2 * j + i;
                    if (a < wlo || a >= whi) continue;
                    const float* sh = stats + (hl * T + a) * 3 * kTile + 4 * (again(lane) >> 5);
                    f32x16 st = scores(qt + i * kTile * G::kPitch, kop);
                    hide(st, block_vis_rows(p, f, kTile * c + (again(lane) & 31), a, nreal));
                    float pr[16];
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const f32x4 m4 = *reinterpret_cast<const f32x4*>(sh + 8 * q4);
                        const f32x4 i4 = *reinterpret_cast<const f32x4*>(sh + kTile + 8 * q4);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            pr[4 * q4 + e] = __builtin_amdgcn_exp2f(fmaf(st[4 * q4 + e], sl2, -m4[e])) * i4[e];
                    }
                    u32x4 wt[2];
                    pack_rows(pr, wt);
                    contract(gt + i * kTile * G::kPitch, wt, dx);
                    const f32x16 dp = scores(gt + i * kTile * G::kPitch, xop);
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const f32x4 d4 = *reinterpret_cast<const f32x4*>(sh + 2 * kTile + 8 * q4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) pr[4 * q4 + e] *= dp[4 * q4 + e] - d4[e];
                    }
                    pack_rows(pr, wt);
                    contract(qt + i * kTile * G::kPitch, wt, dk);
                }
            });
            if (!VS && c < T) {
                set_rowoff(c);
                store_tile_plain<D, NARROW>(dx, 1.f, transit, rowoff, 2, slice(bp.d_vin, h), rows_c, again(lane), dbytes);
            }
        }
        if (c < T) {
            set_rowoff(c);
            u32x4 old[G::kDTiles * 2] = {};
            if (VS) {
                char* dxb = slice(bp.d_vin, g);
                if (bp.acc_x) prefetch_tile<D, NARROW>(old, rowoff, 2, dxb, again(lane), dbytes);
                store_tile<D, NARROW, kBranch>(dx, 1.f, transit, rowoff, 2, dxb, old, bp.acc_x != 0, rows_c, again(lane), dbytes);
            }
            char* dkb = slice(bp.dk, g);
            if (bp.acc_k) prefetch_tile<D, NARROW>(old, rowoff, 1, dkb, again(lane), dbytes);
            store_tile<D, NARROW, kBranch>(dk, p.scale, transit, rowoff, 1, dkb, old, bp.acc_k != 0, rows_c, again(lane), dbytes,
                                  unrope(&p, [&](int r) { return (float)(kTile * c + r); }));
        }
    }
}

// Workgroups per fibre and key/value head.  A fibre's sides are one workgroup's work, 9 products of a pair of tiles (2 for the statistics, 3 for dQ, 4
// for dK and dX), which leaves most of the chip idle on few fibres.  In parts, the query side of eight tiles of a head (5) and the key side of eight
// tiles (4, and the statistics of the rows that see them once more) are workgroups of their own: the longest of them counts, or all together where
// they fill the chip.  One workgroup is resident per CU.
int parts_of(const BwdParams& bp, int tiles) {
    const HopParams& p = bp.hop;
    const int eights = (tiles + kWaves - 1) / kWaves;
    const double units = (double)p.B * p.Hkv * p.fibres, heads = bp.wg_heads;
    double pairs = 0, longest = 0, all = 0;               // in products of one tile against the streamed ones of its eight
    for (int c = eights - 1; c >= 0; --c) {
        pairs += p.causal ? std::min(tiles, kWaves * (c + 1)) : tiles;
        const double seen = p.causal ? pairs : (double)eights * tiles;
        const double key = heads * (2 * seen + 4 * (p.causal ? tiles - kWaves * c : tiles));
        longest = std::max(longest, key);
        all += key;
    }
    all += 5 * heads * pairs;
    // (the factors: measured against this count.  Whole and in parts, us: 8 heads of 128, 1,024 x 4 396 and 182, x 8 404 and 220, x 16 428 and 414, not split; 8 / 2 of 64,
    // 300 x 40 168 and 106, x 80 173 and 186, not split; 8 / 2 of 128, 250 x 20 182 and 130; 8 of 64, 500 x 6 x 2 99 and 83; 32 / 8 of 64, 628 x 2 406 and 214; 12 of
    // 96, 434 142 and 72; 8 of 128 without a mask, 1,000 590 and 231.)
    const double whole = std::ceil(units / 256) * 9 * heads * pairs, split = std::max(1.1 * longest, 1.45 * units * all / 256);
    return split < 0.9 * whole ? eights * (1 + bp.wg_heads) : 1;
}

template <int D, bool VS, bool NARROW, bool ROPE, bool PARTS>
hipError_t launch(const BwdParams& bp, const StreamBwdParams& sp, hipStream_t s) {
    const size_t smem = (size_t)LongGeo<D>::kFixed + (size_t)bp.wg_heads * sp.tiles * 3 * kTile * 4;
    if (smem > (size_t)kStreamMaxLds) return hipErrorInvalidValue;
    const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(mfma_bwd_long_kernel<D, VS, NARROW, ROPE, PARTS>), kStreamMaxLds);
    if (e != hipSuccess) return e;
    const HopParams& p = bp.hop;
    hipLaunchKernelGGL((mfma_bwd_long_kernel<D, VS, NARROW, ROPE, PARTS>), dim3((unsigned)p.Hkv, sp.fibres_lo, (unsigned)p.B * sp.fibres_hi * sp.parts), dim3(64 * kWaves), smem, s, bp, sp);
    return hipGetLastError();
}
template <int D, bool VS, bool NARROW, bool ROPE>
hipError_t launch(const BwdParams& bp, const StreamBwdParams& sp, hipStream_t s) {
    return sp.parts > 1 ? launch<D, VS, NARROW, ROPE, true>(bp, sp, s) : launch<D, VS, NARROW, ROPE, false>(bp, sp, s);
}
template <int D, bool NARROW>
hipError_t launch(const BwdParams& bp, const StreamBwdParams& sp, hipStream_t s) {
    const bool vs = bp.hop.vin_heads != bp.hop.Hq;
    if (bp.hop.rope) return vs ? launch<D, true, NARROW, true>(bp, sp, s) : launch<D, false, NARROW, true>(bp, sp, s);
    return vs ? launch<D, true, NARROW, false>(bp, sp, s) : launch<D, false, NARROW, false>(bp, sp, s);
}

}  // namespace

size_t mfma_backward_long_lds(int32_t n, int32_t heads, int32_t D) {
    return (size_t)(D > 64 ? LongGeo<128>::kFixed : LongGeo<64>::kFixed) + (size_t)heads * ((n + kTile - 1) / kTile) * 3 * kTile * 4;
}

// (wg_heads is not set outside a launch: the first launch of a group takes eight heads at most)
bool mfma_backward_long_in_parts(const BwdParams& bp) {
    const HopParams& p = bp.hop;
    const int64_t lo = p.fibres < 32768 ? p.fibres : 32768, hi = (p.fibres + lo - 1) / lo;
    BwdParams first = bp;
    if (first.wg_heads == 0) first.wg_heads = p.G < 8 ? p.G : 8;
    const int parts = parts_of(first, (p.n + kTile - 1) / kTile);
    return parts > 1 && (int64_t)p.B * hi * parts <= 65535;
}

hipError_t launch_mfma_backward_long(const BwdParams& bp, hipStream_t s) {
    const HopParams& p = bp.hop;
    StreamBwdParams sp;
    sp.q_row = (uint32_t)(p.q.st * 2); sp.k_row = (uint32_t)(p.k.st * 2);
    sp.v_row = (uint32_t)(p.vin.st * 2); sp.o_row = (uint32_t)(bp.d_o.st * 2);
    sp.tiles = (p.n + kTile - 1) / kTile;
    sp.fibres_lo = (uint32_t)(p.fibres < 32768 ? p.fibres : 32768);
    sp.fibres_hi = (uint32_t)((p.fibres + sp.fibres_lo - 1) / sp.fibres_lo);
    if ((int64_t)p.B * sp.fibres_hi > 65535) return hipErrorInvalidValue;
    sp.parts = mfma_backward_long_in_parts(bp) ? parts_of(bp, sp.tiles) : 1;
    return p.D == 128 ? launch<128, false>(bp, sp, s) : p.D == 64 ? launch<64, false>(bp, sp, s)
         : p.D > 64 ? launch<128, true>(bp, sp, s) : launch<64, true>(bp, sp, s);
}

}  // namespace ta
