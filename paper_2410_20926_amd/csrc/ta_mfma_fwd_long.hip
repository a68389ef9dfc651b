// bf16 MFMA per-axis attention forward for long axes on gfx950: one hop of Eq. 4 of arXiv 2410.20926, the keys of a fibre streamed
// 64 at a time with an online softmax.
//
// A workgroup is NW consecutive 32-row query tiles of ONE query head, a wave each (or NW / 4 tiles of four heads that share K and the
// value input).  They walk the same key blocks: every
// wave fetches its share of a block's K and value rows, which enter LDS once for all of them (two buffers and one barrier
// per block, or three and two; the block after next is requested when a block is written, so its rows have a whole block's work to
// arrive).  Per block a wave forms S^T = K Q^T for two 32-key tiles, the softmax of 64 keys at once, O^T += V^T P^T.
//   The weights of each 32-key tile are rounded relative to the row's maximum up to that tile (see below), and the accumulators are
// rescaled only when some row's maximum has grown; the sum of the ROUNDED weights is one dot product per pair of weights.  A tile that
// no row of the query tile sees (half of a diagonal block, padding) is left out; in phases (below) only its value product is.
//   In step, eight waves reach their products, then their softmax, then their products together, and either pipe of a SIMD is idle while
// the other works (32,768 keys of width 128: matrix units busy 37 % of 22.7 M cycles).  On long axes the two halves of the workgroup
// therefore work half a block apart (kPhases): busy 50 % of 16.9 M cycles; the operands of a product are read from LDS a stage ahead, and blocks
// that every row sees whole run without the code for masks.  At width 128 that form takes 256 registers and spills 42 (narrow rows 58); the body
// with masks reloads 8 to 15 of them a block, the one without none.  Value rows lie 16 or 48 banks apart, so that the transposed reads have no bank
// conflicts (half of the LDS cycles before).  The time falls less than the cycles, because the clock falls from 2.33 to about 1.95 GHz.
//   What bounds it: for long axes the power the card may draw (1.04 PFLOP/s; a large bf16 matrix product reaches 1.15), on short ones
// memory and the wait for the first rows.  32 / 8 heads of width 128: 32,768 keys, causal, 9.86 -> 8.46 ms, 16,384 keys, not causal, 4.84 -> 4.08 ms;
// 32 heads of width 64, 8,192 x 2, not causal, 1,567 -> 1,331 us; four tiles: 4,096 keys, not causal, 405 -> 375 us; with the second hop, 128 x 128,
// 200 -> 184 us; 8 heads of 1,024 x 16: 140 -> 116 us, of width 64, 512 x 64: 101 -> 86 us (against a kernel that took 32 keys per barrier and
// rescaled for every tile).  (A reference that moved only when the maximum had passed it by 2^6 took 12 % less in step, with 3 per cent more error.)
#include "ta_mfma_common.h"
#include <algorithm>
#include <type_traits>

namespace ta {
namespace {

using namespace mfma;

constexpr int kKeys = 64;                                 // keys of a block

// Maximum of a lane's and lane ^ 32's value, without a trip through LDS.
__device__ inline float both_halves_max(float x) {
    const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(y[0]), __uint_as_float(y[1]));
}

struct LongParams {
    uint32_t heads;                                       // query heads of a group per workgroup: 1 or 4
    uint32_t qblocks;                                     // workgroups per fibre and set of heads
    uint32_t units;                                       // B * fibres * qblocks * Hkv
    uint32_t q_row, k_row, v_row, o_row;                  // token pitch in bytes
};

// kShort: at most two blocks (n <= 128): both are requested at once and stay, no barrier between them.  kPhases: the two halves of the
// workgroup work half a block apart (see the loop); never with a bit table.
enum Form { kShort, kBlocks, kPhases };
struct Choice { Form form; int waves; };                  // waves per workgroup: 4, or 8 (kPhases: always)
// NARROW: the head is narrower than the D-wide tile; see gather_request.
// 64-wide heads in step: three waves per SIMD, i.e. at most 168 registers (with the 170 that the compiler takes by itself and two waves, 32 / 8 heads
// of 512 x 64: 254 us, here 223).
template <int D, int NW, Form FORM, bool NARROW, bool ROPE>
__global__ __launch_bounds__(64 * NW, D == 64 && FORM != kPhases ? 3 : 2) void mfma_fwd_long_kernel(HopParams p, LongParams lp) {
    using G = Geo<D>;
    constexpr bool SHORT = FORM == kShort, kPhased = FORM == kPhases;
    static_assert(!kPhased || NW == 8, "two sets of four waves");
    // Value rows 16 or 48 banks apart (the four rows of a transposed read on banks of their own), except where blocks of a few hundred keys are
    // worked on in step: there the LDS is not what bounds the kernel, and the smaller buffers are worth 1 to 2 per cent (32 / 8 heads, 512 x 16 of
    // width 128 120.8 us against 122.2; 200 x 64 of width 64 85.0 / 87.1; 16 / 4 heads of width 100, 400 x 30, the other way: 141.4 / 137.5).
    constexpr int kVPitch = FORM == kBlocks ? 2 * D + 16 : 2 * D + 64;
    constexpr int kBlock = kKeys * G::kPitch, kVBlock = kKeys * kVPitch;   // one K, one value block
    constexpr int kBuffers = kPhased ? 3 : 2;
    constexpr int kRows = NW * G::kRowsPerPass;           // rows the workgroup fetches per pass
    constexpr int kMine = kKeys / kRows;                  // passes
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroup -> (unit, head of the group): the heads of a group are 8 workgroup ids apart, i.e. run side by side on one
    // XCD and share their K (and V) rows through its L2
    const uint32_t unit = (blockIdx.z * gridDim.y + blockIdx.y) * 8u + (blockIdx.x & 7u);
    if (unit >= lp.units) return;                         // whole workgroup leaves together
    const int g = (int)(unit % (uint32_t)p.Hkv);
    uint32_t rest = unit / (uint32_t)p.Hkv;
    const int qb = (int)(lp.qblocks - 1 - rest % lp.qblocks);   // heavier blocks (under the causal mask) first
    rest /= lp.qblocks;
    const int64_t f = rest % (uint32_t)p.fibres;
    const int b = (int)(rest / (uint32_t)p.fibres);
    const int tiles = NW / (int)lp.heads;                 // query tiles of the workgroup
    const int h = (int)lp.heads == 1 ? g * p.G + (int)(blockIdx.x >> 3) : g * p.G + 4 * (int)(blockIdx.x >> 3) + (w & 3);
    const int hv = p.vin_heads == p.Hq ? h : g;
    const int n = p.n;
    const uint32_t stride = (uint32_t)p.stride;
    const uint32_t tok0 = (uint32_t)fibre_base_token(f, p.stride, n);
    const char* qbase = reinterpret_cast<const char*>(p.q.p) + ((int64_t)b * p.q.sb + (int64_t)h * p.q.sh) * 2;
    const char* kbase = reinterpret_cast<const char*>(p.k.p) + ((int64_t)b * p.k.sb + (int64_t)g * p.k.sh) * 2;
    const char* vbase = reinterpret_cast<const char*>(p.vin.p) + ((int64_t)b * p.vin.sb + (int64_t)hv * p.vin.sh) * 2;
    char* obase = reinterpret_cast<char*>(p.o.p) + ((int64_t)b * p.o.sb + (int64_t)h * p.o.sh) * 2;

    const int lrow = lane / G::kChunks, lcol = lane % G::kChunks;
    const uint32_t lbyte = lcol * 16;
    const uint32_t dbytes = (uint32_t)p.D * 2;
    const int r32 = lane & 31, hf = lane >> 5;
    float rev[4];
    if constexpr (ROPE) rope_rates(p, lcol, rev);

    const int qt = qb * tiles + (lp.heads == 1 ? w : w >> 2);   // this wave's query tile (past the fibre's end: it only fetches)
    const int vl = (int)min(hop_valid_len(p, b), (int64_t)0x7fffffff);
    const int nreal = (int)tok0 >= vl ? 0 : min(n, (int)(((uint32_t)vl - tok0 + stride - 1) / stride));
    const int qrow = qt * kTile + r32;
    int klo = 0, khi = 0;                                 // this lane's row sees keys [klo, khi)
    if (qrow < nreal) {
        visible_range(qrow, 0, n, p.causal, p.window, klo, khi);
        khi = min(khi, nreal);
    }
    // key blocks that some row of the workgroup sees, and key tiles (half blocks) that some row of this wave's tile sees
    auto keys = [&](int first, int last, int size, int& begin, int& end) {
        int lo, hi, lo2, hi2;
        visible_range(min(first, n - 1), 0, n, p.causal, p.window, lo, hi);
        visible_range(min(last, n - 1), 0, n, p.causal, p.window, lo2, hi2);
        begin = max(lo, 0) / size;
        end = (min(hi2, nreal) + size - 1) / size;
    };
    int jb, je, wb, we;
    keys(qb * tiles * kTile, (qb + 1) * tiles * kTile - 1, kKeys, jb, je);
    keys(qt * kTile, qt * kTile + kTile - 1, kTile, wb, we);
    if (qt * kTile >= nreal) we = wb;
    // A workgroup of nothing but padding writes zeros and takes no block; in phases, where no wave leaves a tile's scores out, it would cost as much as
    // any other (8 sequences of up to 16,713 keys, 8 / 2 heads of width 64, causal: 3,061 us, so 1,868; in step 2,325).
    if (qb * tiles * kTile >= nreal) je = jb;

    // this wave's share of a block: rows w * kRowsPerPass + lrow + i * kRows; rows past the fibre's end: its last one, never visible
    // (Up to 60 features in step spilled a register at three waves per SIMD: 32 heads of 40, 176 x 207 x 2, 357 -> 370 us, now 359)
    constexpr bool kPerLane = D == 64 && NW == 4 && FORM == kBlocks && !ROPE;
    struct Raw { u32x4 v[kMine]; uint32_t mis; };
    const int myrow = w * G::kRowsPerPass + lrow;
    auto request = [&](const char* base, uint32_t pitch, int j, Raw& raw) {
        raw.mis = 0u;
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const uint32_t r = (uint32_t)min(j * kKeys + i * kRows + myrow, n - 1);
            uint32_t mis;
            raw.v[i] = gather_request<NARROW, false, kPerLane>(base, (tok0 + r * stride) * pitch, lbyte, dbytes, mis);
            raw.mis |= mis ? 1u << i : 0u;
        }
    };
    // the same for one block after the other (kPhased: two additions and two minima instead of products): `off` = this lane's first row of
    // the block to be requested next
    auto request_next = [&](const char* base, uint32_t pitch, uint32_t& off, Raw& raw) {
        const uint32_t hop = stride * pitch, last = (tok0 + (uint32_t)(n - 1) * stride) * pitch;
        raw.mis = 0u;
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            uint32_t mis;
            raw.v[i] = gather_request<NARROW, false, kPerLane>(base, min(__builtin_elementwise_add_sat(off, (uint32_t)(i * kRows) * hop), last), lbyte, dbytes, mis);
            raw.mis |= mis ? 1u << i : 0u;
        }
        off = min(__builtin_elementwise_add_sat(off, (uint32_t)kKeys * hop), last);
    };
    auto write = [&](char* block, uint32_t pitch, int j, Raw& raw, bool turn) {
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            u32x4 x = gather_ready<NARROW>(raw.v[i], (raw.mis >> i) & 1u, lbyte, dbytes);
            if (ROPE && turn) x = rope_chunk(x, (float)min(j * kKeys + i * kRows + myrow, n - 1), rev);
            *reinterpret_cast<u32x4*>(block + (uint32_t)(i * kRows + myrow) * pitch + lbyte) = x;
        }
    };
    Raw kr, vr, k2, v2;                                   // (k2: kPhased and SHORT, v2: SHORT only)
    if constexpr (SHORT) { jb = 0; je = (n + kKeys - 1) / kKeys; }
    const uint32_t row0 = tok0 + (uint32_t)min(jb * kKeys + myrow, n - 1) * stride;
    uint32_t koff = row0 * lp.k_row, voff = row0 * lp.v_row;
    if constexpr (kPhased) {
        request_next(kbase, lp.k_row, koff, kr);
        request_next(kbase, lp.k_row, koff, k2);
        request_next(vbase, lp.v_row, voff, vr);
    } else {
        request(kbase, lp.k_row, jb, kr);
        request(vbase, lp.v_row, jb, vr);
    }
    if constexpr (SHORT) {
        request(kbase, lp.k_row, 1, k2);
        request(vbase, lp.v_row, 1, v2);
    }

    // the wave's query rows through LDS into B operands
    u32x4 qop[G::kKSteps];
    {
        char* own = smem + w * (kTile * G::kPitch);
        u32x4 q[G::kPasses];
        uint32_t mis = 0u;
#pragma unroll
        for (int i = 0; i < G::kPasses; ++i)
            q[i] = gather_noted<NARROW, true>(qbase, (tok0 + (uint32_t)min(qt * kTile + i * G::kRowsPerPass + lrow, n - 1) * stride) * lp.q_row, lbyte, dbytes, i, mis);
        gather_ready_all<NARROW>(q, mis, qbase, lp.q_row, lbyte, dbytes);
        if constexpr (ROPE) {
#pragma unroll
            for (int i = 0; i < G::kPasses; ++i) q[i] = rope_chunk(q[i], (float)min(qt * kTile + i * G::kRowsPerPass + lrow, n - 1), rev);
        }
        stage_rows<D>(own + lrow * G::kPitch + lbyte, q);
        lds_wave_sync();
        read_natural<D>(own + r32 * G::kPitch + hf * 16, qop);
    }
    __syncthreads();                                      // the query rows have left LDS
    char* sK = smem;                                      // kBuffers blocks
    char* sV = smem + kBuffers * kBlock;
    write(sK, G::kPitch, jb, kr, true);
    write(sV, kVPitch, jb, vr, false);
    if constexpr (SHORT || kPhased) write(sK + kBlock, G::kPitch, jb + 1, k2, true);
    if constexpr (SHORT) {
        write(sV + kVBlock, kVPitch, 1, v2, false);
    } else if constexpr (kPhased) {
        request_next(kbase, lp.k_row, koff, kr);
        request_next(vbase, lp.v_row, voff, vr);
    } else {
        request(kbase, lp.k_row, jb + 1, kr);
        request(vbase, lp.v_row, jb + 1, vr);
    }
    __syncthreads();

    const uint32_t nat = (uint32_t)(r32 * G::kPitch + hf * 16);
    const uint32_t trn = (uint32_t)((4 * hf + ((lane & 15) >> 2)) * kVPitch + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2);
    const float sl2 = p.scale * kLog2e;
    const bf16x2 ones = __builtin_bit_cast(bf16x2, 0x3f803f80u);
    float m = -INFINITY, l = 0.f;                         // reference value (log2 domain); sum of this lane's weights
    f32x16 ot[G::kDTiles];
#pragma unroll
    for (int t = 0; t < G::kDTiles; ++t) ot[t] = f32x16{};

    auto rescale = [&](float c) {
#pragma unroll
        for (int d = 0; d < G::kDTiles; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) ot[d][r] *= c;
    };
    // masked keys of one or two tiles from number c on; tiles that every row sees whole skip this
    auto mask = [&](auto& st, int c) {
        constexpr int TILES = sizeof(st) / sizeof(st[0]);
        uint32_t vis[TILES], all = 0xffffffffu;
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            vis[t] = range_mask(min(max(klo - kTile * (c + t), 0), kTile), min(max(khi - kTile * (c + t), 0), kTile));
            if (!kPhased && p.mask && qrow < nreal) vis[t] &= table_word(p, (uint32_t)f, qrow, c + t);
            all &= vis[t];
        }
        if (!__all(all == 0xffffffffu)) {
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int r = 0; r < 16; ++r) st[t][r] = ((vis[t] >> (4 * hf + 8 * (r / 4) + (r % 4))) & 1u) ? st[t][r] : -INFINITY;
        }
    };
    // One tile's weights, relative to the row's maximum up to and including that tile, so that the largest is exactly 1:
    // relative to the maximum of both tiles of a block, or to one that lags behind, more of them are rounded (3 per cent more error at
    // 4,096 keys).
    auto weights = [&](const f32x16& st, u32x4 (&pop)[2], float& corr, bool& grows) {
        float mx = st[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, st[r]);
        mx = both_halves_max(mx);
        mx = mx == -INFINITY ? mx : mx * sl2;
        grows = __any(mx > m);                            // (m = -inf: any finite maximum passes it)
        const float top = mx > m ? mx : m;
        corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - top);
        m = top;
        l *= corr;
        const float ref = m == -INFINITY ? 0.f : m;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int r = 8 * s2 + 2 * e;
                const uint32_t pk = pack_bf16x2(__builtin_amdgcn_exp2f(fmaf(st[r], sl2, -ref)), __builtin_amdgcn_exp2f(fmaf(st[r + 1], sl2, -ref)));
                l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), ones, l, false);
                pop[s2][e] = pk;
            }
    };
    // value operand: features 32 d + r32, 16-row step s2 of a tile (see read_transposed)
    auto operand = [&](const char* tile, int d, int s2) {
        const char* a0 = tile + 16 * s2 * kVPitch + 64 * d;
        const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0)));
        const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0 + 8 * kVPitch)));
        return u32x4{lo.x, lo.y, hi.x, hi.y};
    };
    if constexpr (kPhased) {
        // Waves 0-3 and 4-7 work half a block apart, a barrier after each half: while one set forms products (O^T += V^T P^T of block
        // j - 1, then S^T of block j) the other is in the softmax and the staging of its next block, so that the matrix and the
        // vector pipe of a SIMD have one of its two waves each.  In block j's softmax K of block j + 2 and the value input of block j + 1 are
        // written, over blocks j - 1 and j - 2, which the later set has read a phase before; the earlier set reads them two phases later.
        constexpr int kHalf = G::kKSteps / 2;
        using Rows = u32x4[2][kHalf];                     // half the features of a block's two key tiles
        using Values = u32x4[G::kDTiles][2];
        auto key_rows = [&](int slot, int half, Rows& k) {
#pragma unroll
            for (int s = 0; s < kHalf; ++s)
#pragma unroll
                for (int t = 0; t < 2; ++t) k[t][s] = *reinterpret_cast<const u32x4*>(sK + slot * kBlock + t * (kTile * G::kPitch) + nat + 32 * (half * kHalf + s));
        };
        auto score = [&](const Rows& k, int half, f32x16 (&st)[2]) {
#pragma unroll
            for (int s = 0; s < kHalf; ++s)
#pragma unroll
                for (int t = 0; t < 2; ++t) st[t] = mma(k[t][s], qop[half * kHalf + s], st[t]);
        };
        auto value_rows = [&](int slot, int t, Values& v) {
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                for (int d = 0; d < G::kDTiles; ++d) v[d][s2] = operand(sV + slot * kVBlock + t * (kTile * kVPitch) + trn, d, s2);
        };
        auto value = [&](const Values& v, const u32x4 (&w2)[2]) {
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                for (int d = 0; d < G::kDTiles; ++d) ot[d] = mma(v[d][s2], w2[s2], ot[d]);
        };
        // blocks [ia, iz): every row of this wave's tile sees all of their keys (rows past the fibre's end may: they are not stored)
        int ia = je, iz = je;
        if (nreal == n || qt * kTile + kTile <= nreal) {
            int lo, hi, lo2, hi2;
            visible_range(qt * kTile, 0, n, p.causal, p.window, lo, hi);
            visible_range(min(qt * kTile + kTile, n) - 1, 0, n, p.causal, p.window, lo2, hi2);
            ia = min(max((max(lo2, 0) + kKeys - 1) / kKeys, jb), je);
            iz = max(min(min(hi, nreal) / kKeys, je), ia);
        }
        Rows ka;
        key_rows(0, 0, ka);
        int slot = 0;                                     // block j's buffer
        auto step = [&](int j, auto tag) {
            constexpr bool kAll = decltype(tag)::value;
            const int next = slot == 2 ? 0 : slot + 1, after = slot == 0 ? 2 : slot - 1;
            // (both tiles of every block, so that no accumulator is copied where branches meet: one that no row sees gets weights of zero
            // and is left out of the value product)
            Rows kb;
            key_rows(slot, 1, kb);
            f32x16 st[2] = {};
            score(ka, 0, st);
            score(kb, 1, st);
            __builtin_amdgcn_s_setprio(0);
            __syncthreads();
            Values va, vb;
            value_rows(slot, 0, va);
            u32x4 pop[2][2];
            float corr[2];
            bool grows[2];
            if constexpr (!kAll) mask(st, 2 * j);
            weights(st[0], pop[0], corr[0], grows[0]);
            if (grows[0]) rescale(corr[0]);
            weights(st[1], pop[1], corr[1], grows[1]);
            write(sK + after * kBlock, G::kPitch, j + 2, kr, true);   // (past the last block: the fibre's last row, not used)
            write(sV + next * kVBlock, kVPitch, j + 1, vr, false);
            request_next(kbase, lp.k_row, koff, kr);
            request_next(vbase, lp.v_row, voff, vr);
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)                // formed here: they would be moved down to where they are used
                asm volatile("" : "+v"(pop[0][s2]), "+v"(pop[1][s2]));
            __syncthreads();
            __builtin_amdgcn_s_setprio(1);
            value_rows(slot, 1, vb);
            if (kAll || (2 * j >= wb && 2 * j < we)) value(va, pop[0]);
            if (grows[1]) rescale(corr[1]);
            key_rows(next, 0, ka);                        // (past the last block: what is there, not used)
            if (kAll || (2 * j + 1 >= wb && 2 * j + 1 < we)) value(vb, pop[1]);
            slot = next;
        };
        if (w >= 4) __syncthreads();
        int j = jb;
        if (wb >= we) {
            // A wave whose tile lies past the fibre's end or in padding only fetches, with the barriers of the others.  It formed scores and weights of
            // nothing in the longest workgroup of a causal axis, and a tile that is cut off there took every block for a masked one: 8 sequences of
            // 9,000, causal, 4 heads of width 40, 763 us (8,960: 595), so 614; in step 703.  6,600, 4 heads of width 100: 657, so 593; in step 645.
#pragma unroll 1
            for (; j < je; ++j) {
                const int next = slot == 2 ? 0 : slot + 1, after = slot == 0 ? 2 : slot - 1;
                __syncthreads();
                write(sK + after * kBlock, G::kPitch, j + 2, kr, true);
                write(sV + next * kVBlock, kVPitch, j + 1, vr, false);
                request_next(kbase, lp.k_row, koff, kr);
                request_next(vbase, lp.v_row, voff, vr);
                __syncthreads();
                slot = next;
            }
        }
        __builtin_amdgcn_s_setprio(1);
        for (int stop = ia;; stop = je) {
#pragma unroll 1
            for (; j < stop; ++j) step(j, std::false_type{});
            if (j >= je) break;
#pragma unroll 1
            for (; j < iz; ++j) step(j, std::true_type{});
        }
        __builtin_amdgcn_s_setprio(0);
        if (w < 4) __syncthreads();
        __syncthreads();                                  // every block has been read
    } else {
#pragma unroll 1
        for (int j = jb; j < je; ++j) {
            const int slot = (j - jb) & 1;
            if constexpr (!SHORT) {
                if (j + 1 < je) {                             // the other buffer was last read before the last barrier
                    write(sK + (slot ^ 1) * kBlock, G::kPitch, j + 1, kr, true);
                    write(sV + (slot ^ 1) * kVBlock, kVPitch, j + 1, vr, false);
                }
                request(kbase, lp.k_row, j + 2, kr);
                request(vbase, lp.v_row, j + 2, vr);
            }
            // key tiles of the block that some row of the query tile sees: the other half of a diagonal block and padding are left out
            const int first = max(2 * j, wb) - 2 * j, end = min(2 * j + 2, we) - 2 * j;
            if (first < end) {
                // weights of TILES tiles from `first` on, sums and maxima moved on; the first tile's value operands are on their way meanwhile
                u32x4 vop[G::kDTiles][2], pop[2][2];
                float corr[2] = {1.f, 1.f};
                bool grows[2] = {false, false};
                auto values = [&](int t) {
#pragma unroll
                    for (int d = 0; d < G::kDTiles; ++d)
#pragma unroll
                        for (int s2 = 0; s2 < 2; ++s2) vop[d][s2] = operand(sV + slot * kVBlock + t * (kTile * kVPitch) + trn, d, s2);
                };
                auto score = [&](auto tag) {
                    constexpr int TILES = decltype(tag)::value;
                    const char* kt = sK + slot * kBlock + first * (kTile * G::kPitch) + nat;
                    f32x16 st[TILES] = {};
#pragma unroll
                    for (int s = 0; s < G::kKSteps; ++s)
#pragma unroll
                        for (int t = 0; t < TILES; ++t) st[t] = mma(*reinterpret_cast<const u32x4*>(kt + t * (kTile * G::kPitch) + 32 * s), qop[s], st[t]);
                    values(first);
                    mask(st, 2 * j + first);
#pragma unroll
                    for (int t = 0; t < TILES; ++t) weights(st[t], pop[t], corr[t], grows[t]);
                };
                if (end - first == 2) score(std::integral_constant<int, 2>{});
                else score(std::integral_constant<int, 1>{});
#pragma unroll 1
                for (int t = first; t < end; ++t) {           // one body: two would copy the accumulators from one to the other
                    if constexpr (SHORT) {
                        if (grows[0]) rescale(corr[0]);
                    } else if (grows[0]) {                    // (the same: as a call it cost eight waves of 64-wide heads 2 per cent)
#pragma unroll
                        for (int d = 0; d < G::kDTiles; ++d)
#pragma unroll
                            for (int r = 0; r < 16; ++r) ot[d][r] *= corr[0];
                    }
#pragma unroll
                    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                        for (int d = 0; d < G::kDTiles; ++d) ot[d] = mma(vop[d][s2], pop[0][s2], ot[d]);
                    if (t + 1 < end) {
                        values(t + 1);
                        pop[0][0] = pop[1][0]; pop[0][1] = pop[1][1]; corr[0] = corr[1]; grows[0] = grows[1];
                    }
                }
            }
            if (!SHORT) __syncthreads();                      // block j has been read, block j + 1 is complete
        }
        if (SHORT) __syncthreads();                       // every block has been read
    }

    // ---- normalise, round, transpose through LDS, store ----------------------------------------------------
    l += __shfl_xor(l, 32);
    const float inv = l > 0.f ? 1.f / l : 0.f;
    char* own = smem + w * (kTile * G::kPitch);
#pragma unroll
    for (int t = 0; t < G::kDTiles; ++t)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            u32x2 v;
            v.x = pack_bf16x2(ot[t][4 * q4] * inv, ot[t][4 * q4 + 1] * inv);
            v.y = pack_bf16x2(ot[t][4 * q4 + 2] * inv, ot[t][4 * q4 + 3] * inv);
            if (l == 0.f) v = u32x2{0u, 0u};              // a row that sees nothing
            *reinterpret_cast<u32x2*>(own + r32 * G::kPitch + (32 * t + 8 * q4 + 4 * hf) * 2) = v;
        }
    lds_wave_sync();
#pragma unroll
    for (int i = 0; i < G::kPasses; ++i) {
        const int row = qt * kTile + i * G::kRowsPerPass + lrow;
        if (row < n)
            store_row_chunk<NARROW, G::kChunks>(obase, (tok0 + (uint32_t)row * stride) * lp.o_row, own + (i * G::kRowsPerPass + lrow) * G::kPitch + lbyte, lbyte, dbytes);
    }
}

template <int D, int NW, Form FORM, bool NARROW, bool ROPE>
hipError_t launch(const HopParams& p, const LongParams& lp, hipStream_t s) {
    constexpr int smem = (FORM == kPhases ? 3 : 2) * kKeys * (Geo<D>::kPitch + 2 * D + (FORM == kBlocks ? 16 : 64));   // also holds NW query or output tiles
    static_assert(smem >= NW * kTile * Geo<D>::kPitch, "the transit tiles fit");
    if (smem > 64 * 1024) {
        const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(mfma_fwd_long_kernel<D, NW, FORM, NARROW, ROPE>), smem);
        if (e != hipSuccess) return e;
    }
    const uint32_t rows = (lp.units + 7u) / 8u, y = rows < 32768u ? rows : 32768u;
    hipLaunchKernelGGL((mfma_fwd_long_kernel<D, NW, FORM, NARROW, ROPE>), dim3(8u * (uint32_t)p.G / lp.heads, y, (rows + y - 1) / y), dim3(64 * NW), smem, s, p, lp);
    return hipGetLastError();
}
template <int D, bool NARROW, bool ROPE>
hipError_t launch(const HopParams& p, const LongParams& lp, const Choice& how, hipStream_t s) {
    if (how.form == kShort) return launch<D, 4, kShort, NARROW, ROPE>(p, lp, s);
    if (how.waves == 4) return launch<D, 4, kBlocks, NARROW, ROPE>(p, lp, s);
    if constexpr (!ROPE) {
        if (how.form == kPhases) return launch<D, 8, kPhases, NARROW, ROPE>(p, lp, s);
    }
    if constexpr (NARROW || ROPE) return launch<D, 8, kBlocks, NARROW, ROPE>(p, lp, s);
    return hipErrorInvalidValue;                          // (not reached)
}
template <bool ROPE>
hipError_t launch(const HopParams& p, const LongParams& lp, const Choice& how, hipStream_t s) {
    return p.D == 128 ? launch<128, false, ROPE>(p, lp, how, s) : p.D == 64 ? launch<64, false, ROPE>(p, lp, how, s)
         : p.D > 64 ? launch<128, true, ROPE>(p, lp, how, s) : launch<64, true, ROPE>(p, lp, how, s);
}

// Eight query tiles per workgroup (half the K and V rows fetched per query row), in phases or in step, where the axis is long and that leaves a workgroup
// for every CU; else four, in twice the workgroups (one head of width 64, 1,024 keys: 23 against 30 us; 4 / 1 heads of width 128, 2,000 keys: 69 against
// 82).  In phases a wave takes every block that any row of its workgroup sees, and a block with masked keys costs it more; so the keys that a row sees
// (`reach`: the axis, or a window) decide as well, and calls with a bit table stay in step.  Measured on either side (us; 4: four tiles, 8: eight in step,
// p: phases):
//   rows as wide as the tile, from 2,048 positions on: phases, unless a window leaves fewer than 1,280 keys (heads without a group of four 1,536, 64-wide
//     2,048).  Causal, 32 / 8 heads of 128: 2,048 x 16 4 811, p 783; 16,384 2,534, 2,138; two sequences of 16,384, window 64 4 149, p 282; 1,024 740, 755;
//     2,048 1,305, 1,221; 16 heads of 64, window 64 57, 117; 1,024 223, 262; 3,000 521, 530.  Tables of random bits, four sequences of 4,096, not causal:
//     32 / 8 heads of 128 4 1,455, p 1,579; of 64 857, 1,216.  (A table that hides nothing, 16,384, 32 / 8 heads of 128: 5,237, 4,810.)
//   the same, 1,024 to 2,047 positions: phases where the workgroups of eight come out even over the CUs, but not where a causal mask works the four tiles
//     of a group's heads alike, or there are many rounds of unequal workgroups anyway.  8 heads of 128, four sequences of 2,047 4 93, p 80, causal 90, 73;
//     eight of 1,500 109, 115, causal 92, 95; 1,100 x 32, causal, 200, 239; 32 / 8 heads, eight of 1,024 186, 178, causal 121, 134.
//     Lengths of the sequences upset what comes out even (64 drawn calls: causal 13 per cent behind, 64-wide 8, others level): four tiles.
//   narrower rows: eight from 1,024 positions on, in phases from 4,096 positions and 3,000 keys (width up to 64: 1,024) on.  12 heads of 100, causal:
//     3,000 x 8 8 427, p 443; 8,192 x 2 638, 599; 16,384 1,190, 1,078; two sequences of 16,384, window 64 130, 226; 1,024 382, 446; 3,000 865, 870; 8
//     heads of 40, window 512 111, 118; 1,280 196, 187.  Tables of random bits, four of 4,096, 12 heads of 100: 665, 771.
//   encoded rows: eight from 1,024 positions on, never in phases: turning K makes the softmax half of a block the longer one (32 / 8 heads of 128,
//     2,048 x 16: 8 902, p 969).
bool long_params(const HopParams& p, LongParams* lp, Choice* how) {
    if (p.n < 1 || p.D < 8 || p.D > 128 || p.D % 4 != 0 || !mfma_forward_layout_ok(p)) return false;
    // Heads that share K and the value input, four of them per workgroup on the same query tile(s): the waves' work is equal under
    // the causal mask and no wave is without a tile.
    lp->heads = p.G % 4 == 0 && p.vin_heads != p.Hq && p.n > 2 * kKeys ? 4u : 1u;
    const int groups = p.G / (int)lp->heads;
    auto blocks = [&](int waves) { const int rows = waves / (int)lp->heads * kTile; return (p.n + rows - 1) / rows; };
    auto units = [&](int waves) { return (int64_t)p.B * p.fibres * blocks(waves) * p.Hkv; };
    const bool whole = p.D == 64 || p.D == 128;
    const int64_t reach = p.window > 0 ? std::min<int64_t>(p.n, p.causal ? p.window : 2 * (int64_t)p.window - 1) : p.n;
    const int64_t wgs = units(8) * groups;
    const bool eight = p.n >= 1024 && wgs >= 256;
    bool phases = eight && !p.rope && !p.mask;
    if (!whole) phases = phases && p.n >= 4096 && reach >= (p.D > 64 ? 3000 : 1024);
    else if (p.n >= 2048) phases = phases && reach >= (p.D == 64 ? 2048 : lp->heads == 4 ? 1280 : 1536);
    else phases = phases && reach == p.n && !p.valid_lens && (wgs % 256 == 0 || wgs % 256 >= 192) && (!p.causal || (lp->heads == 1 && wgs <= (p.D == 128 ? 768 : 256)));
    how->form = p.n <= 2 * kKeys ? kShort : phases ? kPhases : kBlocks;
    how->waves = phases || (eight && (!whole || p.rope)) ? 8 : 4;
    lp->qblocks = (uint32_t)blocks(how->waves);
    const int64_t n_units = units(how->waves);
    if (n_units <= 0 || n_units > 0x7ffffff0LL || p.G > (1 << 19)) return false;
    lp->units = (uint32_t)n_units;
    lp->q_row = (uint32_t)(p.q.st * 2); lp->k_row = (uint32_t)(p.k.st * 2);
    lp->v_row = (uint32_t)(p.vin.st * 2); lp->o_row = (uint32_t)(p.o.st * 2);
    return true;
}

}  // namespace

bool mfma_forward_long_feasible(const HopParams& p) {
    LongParams lp;
    Choice how;
    return long_params(p, &lp, &how);
}

const char* mfma_forward_long_form(const HopParams& p) {
    LongParams lp;
    Choice how;
    if (!long_params(p, &lp, &how)) return "unsupported";
    return how.form == kShort ? "two_blocks" : how.form == kPhases ? "eight_tiles_in_phases" : how.waves == 8 ? "eight_tiles_in_step" : "four_tiles_in_step";
}

hipError_t launch_mfma_forward_long(const HopParams& p, hipStream_t s) {
    LongParams lp;
    Choice how;
    if (!long_params(p, &lp, &how)) return hipErrorInvalidValue;
    return p.rope ? launch<true>(p, lp, how, s) : launch<false>(p, lp, how, s);
}

}  // namespace ta
