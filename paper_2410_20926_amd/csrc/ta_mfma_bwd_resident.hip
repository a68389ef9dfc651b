// bf16 MFMA backward for axes of two to four tiles (32 < n <= 128), gfx950.  The derivative itself is that of
// ta_mfma_bwd.hip.
//
// The whole fibre stays in LDS.  A workgroup is two waves per 32-row tile and works through the query heads of a key/value
// head one after the other; the fibre's K, value, Q and dO tiles are staged once per head, and nothing is computed twice:
//   query side   the two waves of tile t form S^T and dP^T of query tile t, each against every other key tile; they
//                exchange the row statistics (max, sum, sum of P o dP), so that P and dS are exact; each forms its key
//                tiles' share of dQ_t; P and dS then go, as bf16 rows, over the value and K tiles that nobody needs any more.
//   key side     tile t is now key tile t: each of its waves forms one half of the features of dX_t and dK_t from the
//                rows of P and dS and the transposed dO and Q tiles.
// dK, and dX of a per-group value input, add up over the heads in registers: no sum over heads through LDS, no atomics, one
// rounding.  While a head is worked on, the next head's rows (or the next fibre's: a workgroup takes every
// gridDim.x-th one) are on their way into registers, half a tile per wave and tensor.
//
// A request is waited for with a count of what was issued behind it, loads and stores alike, so two things stand between the rows on their way and
// their use: a store that may or may not have been issued, after which every wait is for all of them (stores go through the buffer's bounds check
// instead of a branch, row_buffer), and a spilled value, whose reload waits for every row requested before it (what depends on the lane is formed anew
// wherever it is used; narrow 128-wide instantiations had 12 to 29 spilled registers, now 0 to 4).  32 / 8 heads of 96, 13 x 52 x 71, hops of 1,078 / 800 ->
// 866 / 584 us, of 100, 64 x 64 x 32, 1,965 -> 1,351; whole rows of 128 features, 128 x 128, 193 / 183 -> 189 / 175.
//
// What bounds it: memory, and seven barriers per head of which one workgroup per CU (width 128, n > 64) hides little (LDS active 30 % of
// the time, 41 % of that in bank conflicts, matrix units busy 9 %).  The
// blocked kernel, which it replaces up to 128, gathers every tile again at each visit, waits for each, and forms S and dP up to
// four times.  128 x 128 tokens, 32 / 8 heads of width 128, causal: hops of 437 / 395 us -> 189 / 175 us;
// 100 x 100, batch 2, 12 heads of width 96: 407 -> 218 us; 64 x 64 x 32, 32 / 8 heads: the two-tile kernel's 1522 / 1544 us -> 1365 / 1185 us
// (5.3 and 4.8 TB/s).  A first form with one wave per tile and 512 registers took 450 us at 128 x 128: it spilled, and a
// reload waits for every row requested before it.
#include "ta_mfma_bwd_common.h"
#include <type_traits>

namespace ta {
namespace {

using namespace mfma;

template <int D, int TM>
struct Resident {
    static constexpr int kHalf = D / 2;                                       // features of one wave's share of an output
    static constexpr int kHT = kHalf / 32;                                    // 32-feature tiles of it
    static constexpr int kOutLanes = kHalf / 8;                               // 16-byte chunks of its row
    static constexpr int kOutRows = 64 / kOutLanes;                           // rows of one wave-wide store
    static constexpr int kOut = kTile / kOutRows;                             // stores per lane
    static constexpr int kFPitch = kHalf * 4 + 16;                            // bytes, a row of the epilogue's fp32 transit
    static constexpr int kBuf = kTile * Geo<D>::kPitch;                       // a Q or dO tile
    static constexpr int kWPitch = TM * kTile * 2 + 16;                       // bytes, a row of P or dS
    static constexpr int kMax = kTile * (kWPitch > kFPitch ? kWPitch : kFPitch);
    static constexpr int kRegion = kBuf > kMax ? kBuf : kMax;                 // a K or value tile, 32 rows of dS or P, or the transit
    static constexpr int kStats = 2 * 3 * kTile * 4;                          // both waves' max, sum, sum of P o dP
    static constexpr int kTileBytes = 2 * kBuf + 2 * kRegion + kStats;        // LDS per tile
};

// MODE: what the heads of a group share.  kOne: a group is one head, nothing is shared or summed; kHeads: K; kGroup: K and the
// value input (the value input is V).  NARROW: the head is narrower than the D-wide tile; see gather_request.
enum : int { kOne, kHeads, kGroup };
template <int D, int TM, int MODE, bool NARROW, bool ROPE>
__global__ __launch_bounds__(128 * TM, 2) void mfma_bwd_resident_kernel(BwdParams bp, StreamBwdParams sp, uint32_t units) {
    using G = BGeo<D>;
    using R = Resident<D, TM>;
    constexpr bool VS = MODE == kGroup;
    constexpr int kMine = G::kPasses / 2;                 // loads per lane of this wave's half of a tile
    constexpr int kCT = TM / 2;                           // key tiles per wave on the query side
    const HopParams& p = bp.hop;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = wave >> 1, s = wave & 1;                // tile; which of its two waves
    const int T = sp.tiles, n = p.n;                      // blockDim.x = 128 T
    char* sK = smem;
    char* sX = sK + T * R::kRegion;
    char* sQ = sX + T * R::kRegion;
    char* sG = sQ + T * R::kBuf;
    float* stats = reinterpret_cast<float*>(sG + T * R::kBuf) + w * (R::kStats / 4);
    char* transit = (s ? sK : sX) + w * R::kRegion;

    const uint32_t dbytes = (uint32_t)p.D * 2;
    const uint32_t stride = (uint32_t)p.stride;
    const int rows_t = min(kTile, n - kTile * w);
    const float sl2 = p.scale * kLog2e;

    // key tiles [cb, ce) that some row of query tile a sees
    auto key_tiles = [&](int a, int& cb, int& ce) {
        int lo, hi, lo2, hi2;
        visible_range(kTile * a, 0, n, p.causal, p.window, lo, hi);
        visible_range(min(kTile * a + kTile - 1, n - 1), 0, n, p.causal, p.window, lo2, hi2);
        cb = max(lo, 0) / kTile;
        ce = (min(hi2, n) + kTile - 1) / kTile;
    };
    bool sees[kCT], seen[TM];                             // query tile w sees key tile 2 i + s; query tile i sees key tile w
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        int cb, ce;
        key_tiles(min(i, T - 1), cb, ce);
        seen[i] = i < T && w >= cb && w < ce;
        key_tiles(w, cb, ce);
        if (i < kCT) sees[i] = 2 * i + s >= cb && 2 * i + s < ce && 2 * i + s < T;
    }

    struct Where { int b, g; int64_t f; uint32_t tok0; };
    auto where = [&](uint32_t u) {
        if constexpr (NARROW) {                           // each XCD takes a contiguous run of (fibre, head) pairs, see workgroup_xy
            if (gridDim.x % 8u == 0u) u = xcd_order(u, units, kLongestRun);
        }
        Where x;
        x.g = (int)(u % (uint32_t)p.Hkv);
        const uint32_t rest = u / (uint32_t)p.Hkv;
        x.f = rest % (uint32_t)p.fibres;
        x.b = (int)(rest / (uint32_t)p.fibres);
        x.tok0 = (uint32_t)fibre_base_token(x.f, p.stride, n);
        return x;
    };
    // This wave's half of tile w (rows past the fibre's end: its last row, masked in the softmax and never stored).
    // `once`: nobody asks for these rows again (K and a per-group value input are asked for by every head).
    // The rows are only requested here; `ready` turns what has come into this lane's chunks (see gather_request: NARROW rows start
    // 8 bytes into an aligned unit or on one, `mis` has a bit per row).
    enum : int { kRawQ, kRawG, kRawX, kRawK };
    struct Raw { u32x4 v[kMine]; };
    uint32_t misaligned = 0u;                             // NARROW: a bit per requested row, 4 bits per tensor
    // What depends on the lane is formed anew wherever it is used, from a copy of the lane's number that the compiler cannot look
    // through: kept over the loop it would be spilled, and a reload waits for every row requested before it.  64-wide tiles have more room: narrow or
    // encoded rows form it once per head (32 / 8 heads of 40, 9 x 38 x 42 x 8, 803 -> 754 us), whole rows of three and four tiles keep it (8 / 2 heads, 50 x 70, 23.3 -> 22.2 us
    // against new row addresses, 32 / 8, 100 x 200, 176 -> 168; encoded, 128 x 128, 116.5 before any was formed anew, 117.9 once per head, 104.0), of two all but row addresses (kept, they take 27 registers more and a wave per SIMD: 32 / 8 heads, 500 x 40, 113 against 145).
    int head_lane = threadIdx.x & 63;
    auto fresh_lane = [&]() {
        int l = head_lane;
        if (D == 128 || (TM == 2 && !(NARROW || ROPE))) asm volatile("" : "+v"(l));
        return l;
    };
    // (Whole 128-wide rows with a value input per head of a group have the registers to keep it for the exchanges: 32 / 8 heads, 18 x 81 x 66 x 3, 4,615 -> 4,704 us with it formed
    // anew everywhere, 4,609 now; 128 x 128 196 -> 193 -> 191; 18 hops 0.991 -> 0.983.)
    auto kept_lane = [&]() { return D == 128 && (NARROW || ROPE || MODE != kHeads) ? fresh_lane() : head_lane; };
    auto gather = [&](auto once, auto which, const Tensor& t, const Where& x, int head, uint32_t pitch, Raw& raw) {
        const char* base = reinterpret_cast<const char*>(t.p) + ((int64_t)x.b * t.sb + (int64_t)head * t.sh) * 2;
        const int l = fresh_lane(), row = l / G::kChunks;
        const uint32_t lbyte = (uint32_t)(l % G::kChunks) * 16;
        if constexpr (NARROW) misaligned &= ~(15u << (4 * decltype(which)::value));
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const uint32_t rr = (uint32_t)min(kTile * w + (s * kMine + i) * G::kRowsPerPass + row, n - 1);
            uint32_t mis;
            raw.v[i] = gather_request<NARROW, decltype(once)::value>(base, (x.tok0 + rr * stride) * pitch, lbyte, dbytes, mis);
            if constexpr (NARROW) misaligned |= (mis >> 3) << (4 * decltype(which)::value + i);
        }
    };
    auto put = [&](char* tile, const Raw& raw) {
        const int l = kept_lane();
        const uint32_t stg = (uint32_t)((s * kMine * G::kRowsPerPass + l / G::kChunks) * G::kPitch + (l % G::kChunks) * 16);
#pragma unroll
        for (int i = 0; i < kMine; ++i) *reinterpret_cast<u32x4*>(tile + stg + i * G::kRowsPerPass * G::kPitch) = raw.v[i];
    };
    auto ready = [&](auto which, Raw& raw) {
        if constexpr (NARROW) {
            const uint32_t lbyte = (uint32_t)(fresh_lane() % G::kChunks) * 16;
#pragma unroll
            for (int i = 0; i < kMine; ++i) raw.v[i] = gather_ready<NARROW>(raw.v[i], (misaligned >> (4 * decltype(which)::value + i)) & 1u, lbyte, dbytes);
        }
    };
    auto encode = [&](auto which, Raw& raw) {
        ready(which, raw);
        if constexpr (ROPE) {
            const int l = fresh_lane(), row = l / G::kChunks;
            float rev[4];
            rope_rates(p, l % G::kChunks, rev);
#pragma unroll
            for (int i = 0; i < kMine; ++i) raw.v[i] = rope_chunk(raw.v[i], (float)min(kTile * w + (s * kMine + i) * G::kRowsPerPass + row, n - 1), rev);
        }
    };
    // A finished half of an output tile: acc[t][r] = (row r32, feature kHalf s + 32 t + 8 (r / 4) + 4 hf + r % 4), turned in LDS,
    // turned back when the hop encodes positions, added to the previous contents, rounded, stored.
    // (Rows past the fibre's end are loaded as its last row and never stored.)
    auto out_lane = [&](int& orow, uint32_t& obyte) {
        const int l = fresh_lane();
        orow = l / R::kOutLanes;
        obyte = (uint32_t)(s * R::kHalf * 2 + (l % R::kOutLanes) * 16);
    };
    auto out_offset = [&](uint32_t tok0, int row, uint32_t pitch) { return (tok0 + (uint32_t)(kTile * w + row) * stride) * pitch; };
    auto previous = [&](const char* base, uint32_t tok0, uint32_t pitch, u32x4 (&old)[R::kOut]) {
        int orow;
        uint32_t obyte;
        out_lane(orow, obyte);
#pragma unroll
        for (int i = 0; i < R::kOut; ++i) {
            const uint32_t off = out_offset(tok0, min(i * R::kOutRows + orow, rows_t - 1), pitch);
            if constexpr (!NARROW) {
                old[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (off + obyte)));
            } else {                                      // a chunk that would pass the end of the row: the row's last 16 bytes (see `finish`)
                old[i] = *reinterpret_cast<const u32x4*>(base + (off + min(obyte, dbytes - 16)));
            }
        }
    };
    auto finish = [&](auto turn, const f32x16 (&acc)[R::kHT], float mult, char* base, uint32_t tok0, uint32_t pitch, const u32x4 (&old)[R::kOut], bool add) {
        int orow;
        uint32_t obyte;
        out_lane(orow, obyte);
        const int la = kept_lane(), r32 = la & 31, hf = la >> 5;
        lds_wave_sync();
#pragma unroll
        for (int t = 0; t < R::kHT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4*>(transit + r32 * R::kFPitch + (32 * t + 8 * q + 4 * hf) * 4) =
                    f32x4{acc[t][4 * q] * mult, acc[t][4 * q + 1] * mult, acc[t][4 * q + 2] * mult, acc[t][4 * q + 3] * mult};
        lds_wave_sync();
        float y[R::kOut][8];
#pragma unroll
        for (int i = 0; i < R::kOut; ++i) {
            const char* at = transit + (i * R::kOutRows + orow) * R::kFPitch + 2 * (obyte - (uint32_t)(s * R::kHalf * 2));
            const f32x4 x0 = *reinterpret_cast<const f32x4*>(at), x1 = *reinterpret_cast<const f32x4*>(at + 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) { y[i][e] = x0[e]; y[i][4 + e] = x1[e]; }
        }
        if constexpr (ROPE && decltype(turn)::value) {
            float orev[4], c[4], sn[4];
            rope_rates(p, (int)(obyte / 16), orev);
#pragma unroll
            for (int i = 0; i < R::kOut; ++i) {
                rope_sincos((float)(kTile * w + i * R::kOutRows + orow), orev, c, sn);
                rope_apply_f32<true>(y[i], c, sn);
            }
        }
        if (add) {
            const bool tail = NARROW && obyte + 8 == dbytes;   // this lane has the row's last 8 bytes: the second half of what it asked for
#pragma unroll
            for (int i = 0; i < R::kOut; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t o = NARROW && e < 2 ? (tail ? old[i][e + 2] : old[i][e]) : old[i][e];
                    y[i][2 * e] += bf16_lo(o);
                    y[i][2 * e + 1] += bf16_hi(o);
                }
        }
        const __amdgpu_buffer_rsrc_t to = row_buffer(base);
#pragma unroll
        for (int i = 0; i < R::kOut; ++i)
            buffer_store_chunk<NARROW>(to, out_offset(tok0, i * R::kOutRows + orow, pitch), i * R::kOutRows + orow < rows_t, obyte, dbytes,
                                       u32x4{pack_bf16x2(y[i][0], y[i][1]), pack_bf16x2(y[i][2], y[i][3]), pack_bf16x2(y[i][4], y[i][5]), pack_bf16x2(y[i][6], y[i][7])}, dbytes % 16 == 0);
    };

    Where at = where(blockIdx.x);
    Raw qraw, graw, xraw, kraw;
    using Once = std::bool_constant<!NARROW>;
    using Again = std::false_type;
    using IsQ = std::integral_constant<int, kRawQ>;
    using IsG = std::integral_constant<int, kRawG>;
    using IsX = std::integral_constant<int, kRawX>;
    using IsK = std::integral_constant<int, kRawK>;
    using Turn = std::true_type;
    using AsIs = std::false_type;
    // The next head's own rows are requested as soon as this head's are in LDS; those that the heads share, mostly in L2, near
    // the head's end, when there are registers again.  Always issued: requests under a branch that live across the loop were all spilled.
    auto request_own = [&](const Where& x, int head) {
        gather(Once{}, IsQ{}, p.q, x, head, sp.q_row, qraw);
        gather(Once{}, IsG{}, bp.d_o, x, head, sp.o_row, graw);
        if constexpr (!VS) gather(Once{}, IsX{}, p.vin, x, head, sp.v_row, xraw);
        if constexpr (MODE == kOne) gather(Once{}, IsK{}, p.k, x, x.g, sp.k_row, kraw);
    };
    auto request_shared = [&](const Where& x) {
        if constexpr (MODE != kOne) gather(Again{}, IsK{}, p.k, x, x.g, sp.k_row, kraw);
        if constexpr (VS) gather(Again{}, IsX{}, p.vin, x, x.g, sp.v_row, xraw);
    };
    request_shared(at);
    request_own(at, at.g * p.G);
    // (No wait for all of them here: a workgroup's first head is staged tensor by tensor as they come.  With one, which was to leave the loop's waits nothing but
    // the loop's own requests and stores to count, calls of one or two pairs per workgroup took 2 to 8 per cent longer and none less.)
#pragma unroll 1
    for (uint32_t u = blockIdx.x; u < units; u += gridDim.x) {
        f32x16 dk[R::kHT], dx[R::kHT];
#pragma unroll
        for (int t = 0; t < R::kHT; ++t) { dk[t] = f32x16{}; dx[t] = f32x16{}; }
        const Where nx = where(u + gridDim.x < units ? u + gridDim.x : u);   // the last fibre requests itself again
        const uint32_t vl = (uint32_t)hop_valid_len(p, at.b);
        const int nreal = at.tok0 >= vl ? 0 : (int)min((uint32_t)n, (vl - at.tok0 + stride - 1) / stride);
        char* dkb = reinterpret_cast<char*>(bp.dk.p) + ((int64_t)at.b * bp.dk.sb + (int64_t)at.g * bp.dk.sh) * 2;
#pragma unroll 1
        for (int hl = 0; hl < (MODE == kOne ? 1 : p.G); ++hl) {
            const int h = at.g * p.G + hl, hv = VS ? at.g : h;
            const bool last_head = MODE == kOne || hl + 1 == p.G;
            if (D == 64 && (NARROW || (ROPE && TM == 2))) asm volatile("" : "+v"(head_lane));
            const int l_ = fresh_lane(), r32 = kept_lane() & 31, hf = kept_lane() >> 5;
            const int qr = kTile * w + r32;               // this lane's query row
            const uint32_t nat = (uint32_t)((l_ & 31) * G::kPitch + (l_ >> 5) * 16);
            const uint32_t trow = (uint32_t)(4 * (l_ >> 5) + ((l_ & 15) >> 2)), tcol = (uint32_t)(16 * ((l_ >> 4) & 1) + 4 * (l_ & 3)) * 2;
            const uint32_t trn = trow * G::kPitch + tcol;
            encode(IsK{}, kraw);
            put(sK + w * R::kRegion, kraw);
            ready(IsX{}, xraw);
            put(sX + w * R::kRegion, xraw);
            encode(IsQ{}, qraw);
            put(sQ + w * R::kBuf, qraw);
            ready(IsG{}, graw);
            put(sG + w * R::kBuf, graw);
            request_own(last_head ? nx : at, last_head ? nx.g * p.G : h + 1);
            char* dqb = reinterpret_cast<char*>(bp.dq.p) + ((int64_t)at.b * bp.dq.sb + (int64_t)h * bp.dq.sh) * 2;
            __syncthreads();                              // (1) every tile is staged

            // ---- query side: S^T and dP^T of query tile w against this wave's key tiles --------------------
            f32x16 st[kCT], dp[kCT];
            float mx = -INFINITY;
#pragma unroll
            for (int i = 0; i < kCT; ++i) {
                st[i] = f32x16{}; dp[i] = f32x16{};
                if (sees[i]) {
                    const char* kt = sK + (2 * i + s) * R::kRegion + nat;
                    const char* xt = sX + (2 * i + s) * R::kRegion + nat;
#pragma unroll
                    for (int k = 0; k < G::kKSteps; ++k)
                        st[i] = mma(*reinterpret_cast<const u32x4*>(kt + 32 * k), *reinterpret_cast<const u32x4*>(sQ + w * R::kBuf + nat + 32 * k), st[i]);
#pragma unroll
                    for (int k = 0; k < G::kKSteps; ++k)
                        dp[i] = mma(*reinterpret_cast<const u32x4*>(xt + 32 * k), *reinterpret_cast<const u32x4*>(sG + w * R::kBuf + nat + 32 * k), dp[i]);
                    uint32_t vis = block_vis_keys(p, at.f, qr, 2 * i + s, nreal);
                    if (!__all(vis == 0xffffffffu)) {     // masked keys; a block that every row sees whole skips this
                        vis >>= 4 * hf;
#pragma unroll
                        for (int r = 0; r < 16; ++r) st[i][r] = ((vis >> (8 * (r / 4) + (r % 4))) & 1u) ? st[i][r] : -INFINITY;
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, st[i][r]);
                }
            }
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float own = mx == -INFINITY ? 0.f : mx * sl2;   // weights relative to this wave's own maximum first
            float l = 0.f, dn = 0.f;
#pragma unroll
            for (int i = 0; i < kCT; ++i)
                if (sees[i]) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float e = __builtin_amdgcn_exp2f(fmaf(st[i][r], sl2, -own));
                        st[i][r] = e;
                        l += e;
                        dn += e * dp[i][r];
                    }
                }
            l += __shfl_xor(l, 32);
            dn += __shfl_xor(dn, 32);
            if (hf == 0) { stats[(3 * s) * kTile + r32] = mx; stats[(3 * s + 1) * kTile + r32] = l; stats[(3 * s + 2) * kTile + r32] = dn; }
            __syncthreads();                              // (2) both waves' statistics are there
            float f, delta;                               // what the weights are multiplied by; rowsum(P o dP)
            {
                const float m2 = stats[3 * (1 - s) * kTile + r32], l2 = stats[(3 * (1 - s) + 1) * kTile + r32], d2 = stats[(3 * (1 - s) + 2) * kTile + r32];
                const float oth = m2 == -INFINITY ? 0.f : m2 * sl2, top = fmaxf(mx, m2) == -INFINITY ? 0.f : fmaxf(mx, m2) * sl2;
                const float c1 = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(own - top), c2 = m2 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(oth - top);
                const float lt = l * c1 + l2 * c2;
                const float inv = lt > 0.f ? 1.f / lt : 0.f;
                f = c1 * inv;
                delta = (dn * c1 + d2 * c2) * inv;
            }
            u32x4 pop[kCT][2], dsop[kCT][2];
#pragma unroll
            for (int i = 0; i < kCT; ++i) {
                float pw[16], ds[16];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    pw[r] = st[i][r] * f;
                    ds[r] = pw[r] * (dp[i][r] - delta);
                }
                pack_rows(pw, pop[i]);
                pack_rows(ds, dsop[i]);
            }
            f32x16 dq[G::kDTiles];                        // this wave's key tiles' share, every feature
#pragma unroll
            for (int t = 0; t < G::kDTiles; ++t) dq[t] = f32x16{};
#pragma unroll
            for (int i = 0; i < kCT; ++i)
                if (sees[i]) {
                    u32x4 kT[G::kDTiles][2];
                    read_transposed<D>(sK + (2 * i + s) * R::kRegion + trn, kT);
#pragma unroll
                    for (int t = 0; t < G::kDTiles; ++t)
#pragma unroll
                        for (int s2 = 0; s2 < 2; ++s2) dq[t] = mma(kT[t][s2], dsop[i][s2], dq[t]);
                }
            __syncthreads();                              // (3) the K and value tiles have been read by everyone
#pragma unroll
            for (int i = 0; i < kCT; ++i)                 // rows of P and dS (32 w + r32, keys 32 c ..) over them
                if (sees[i]) {
                    const uint32_t o = (uint32_t)(w * R::kRegion + r32 * R::kWPitch + (32 * (2 * i + s) + 4 * hf) * 2);
#pragma unroll
                    for (int s2 = 0; s2 < 2; ++s2) {
                        *reinterpret_cast<u32x2*>(sX + o + 32 * s2) = u32x2{pop[i][s2].x, pop[i][s2].y};
                        *reinterpret_cast<u32x2*>(sX + o + 32 * s2 + 16) = u32x2{pop[i][s2].z, pop[i][s2].w};
                        *reinterpret_cast<u32x2*>(sK + o + 32 * s2) = u32x2{dsop[i][s2].x, dsop[i][s2].y};
                        *reinterpret_cast<u32x2*>(sK + o + 32 * s2 + 16) = u32x2{dsop[i][s2].z, dsop[i][s2].w};
                    }
                }
            __syncthreads();                              // (4) P and dS are complete

            // ---- key side: this wave's features of dX_w^T += dO_a^T P_aw and dK_w^T += Q_a^T dS_aw ----------
            if (!VS) {
#pragma unroll
                for (int t = 0; t < R::kHT; ++t) dx[t] = f32x16{};
            }
            if (MODE == kOne) {
#pragma unroll
                for (int t = 0; t < R::kHT; ++t) dk[t] = f32x16{};
            }
            auto contract = [&](const char* weights, const char* tile, int a, f32x16 (&acc)[R::kHT]) {
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    auto pair = [&](const char* a0, int pitch) {
                        const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0)));
                        const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0 + 8 * pitch)));
                        return u32x4{lo.x, lo.y, hi.x, hi.y};
                    };
                    const u32x4 wt = pair(weights + a * R::kRegion + (16 * s2 + trow) * R::kWPitch + 64 * w + tcol, R::kWPitch);
#pragma unroll
                    for (int t = 0; t < R::kHT; ++t)
                        acc[t] = mma(pair(tile + a * R::kBuf + trn + 16 * s2 * G::kPitch + 64 * (s * R::kHT + t), G::kPitch), wt, acc[t]);
                }
            };
#pragma unroll
            for (int a = 0; a < TM; ++a)
                if (seen[a]) {
                    contract(sX, sG, a, dx);
                    contract(sK, sQ, a, dk);
                }
            char* dxb = reinterpret_cast<char*>(bp.d_vin.p) + ((int64_t)at.b * bp.d_vin.sb + (int64_t)hv * bp.d_vin.sh) * 2;
            u32x4 old[R::kOut] = {}, oldk[R::kOut] = {};
            if (bp.accumulate) {
                previous(dqb, at.tok0, sp.q_row, old);
                if (last_head) previous(dkb, at.tok0, sp.k_row, oldk);
            }
            __syncthreads();                              // (5) nobody reads this head's tiles any more
            // the partner's half of dQ's features goes to the partner (its transit area), lane by lane
            {
                char* there = (s ? sX : sK) + w * R::kRegion + l_ * 16;
#pragma unroll
                for (int t = 0; t < R::kHT; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x16 &x0 = dq[t], &x1 = dq[R::kHT + t];
                        const f32x4 v0 = {x0[4 * q], x0[4 * q + 1], x0[4 * q + 2], x0[4 * q + 3]}, v1 = {x1[4 * q], x1[4 * q + 1], x1[4 * q + 2], x1[4 * q + 3]};
                        *reinterpret_cast<f32x4*>(there + (4 * t + q) * 1024) = s ? v0 : v1;
                    }
            }
            request_shared(last_head ? nx : at);
            __syncthreads();                              // (6) both shares are there
            f32x16 mine[R::kHT];
#pragma unroll
            for (int t = 0; t < R::kHT; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(transit + l_ * 16 + (4 * t + q) * 1024);
#pragma unroll
                    for (int e = 0; e < 4; ++e) mine[t][4 * q + e] = (s ? dq[R::kHT + t][4 * q + e] : dq[t][4 * q + e]) + v[e];
                }
            finish(Turn{}, mine, p.scale, dqb, at.tok0, sp.q_row, old, bp.accumulate != 0);
            if (!VS || last_head) finish(AsIs{}, dx, 1.f, dxb, at.tok0, sp.v_row, old, false);
            if (last_head) finish(Turn{}, dk, p.scale, dkb, at.tok0, sp.k_row, oldk, bp.accumulate != 0);
            __syncthreads();                              // (7) the areas of transit are free for the next head's tiles
        }
        at = nx;
    }
}

template <int D, int TM, int MODE, bool NARROW, bool ROPE>
hipError_t launch_resident(const BwdParams& bp, hipStream_t s) {
    const HopParams& p = bp.hop;
    StreamBwdParams sp;
    sp.q_row = (uint32_t)(p.q.st * 2); sp.k_row = (uint32_t)(p.k.st * 2);
    sp.v_row = (uint32_t)(p.vin.st * 2); sp.o_row = (uint32_t)(bp.d_o.st * 2);
    sp.tiles = (p.n + kTile - 1) / kTile;
    sp.fibres_lo = sp.fibres_hi = 0;
    const int64_t units = (int64_t)p.B * p.Hkv * p.fibres;
    if (units <= 0 || units > 0x7fffffffLL || p.n > TM * kTile) return hipErrorInvalidValue;
    const size_t smem = (size_t)sp.tiles * Resident<D, TM>::kTileBytes;
    // as many workgroups as are resident at once (8 waves of up to 256 registers per CU, 12 of the smallest instantiation's 168):
    // each walks its share of the fibres, but for narrow rows below
    const int by_lds = (int)((size_t)kStreamMaxLds / smem), by_regs = (D == 64 && TM == 2 ? 6 : 4) / sp.tiles;
    const int per_cu = by_lds < by_regs ? by_lds : by_regs;
    const int64_t most = 256 * (per_cu < 1 ? 1 : per_cu);
    // Narrow rows share lines with the neighbouring heads' rows, which find them in L2 only as long as their workgroups keep step.  Workgroups that walk a
    // long share drift apart by more than L2 holds (32 heads of 100, 64 x 64 x 32: 1.63 times the algorithmic bytes read, 1.25 in shares of four), so where there is enough for it they
    // take four (fibre, head) pairs each and are replaced in order: 3,000 -> 1,950 us, of 96 2,130 -> 1,700, of 40 1,440 -> 794; 8 of 36,
    // 60 x 238 x 9 x 2, 507 -> 355; at the lower ends of the rule 32 of 48, 63 x 19 x 9 x 2, 196 -> 139, 12 of 100, 251 x 50 x 4, 325 -> 293.
    // With less it costs a start that nothing hides more often than it gains (long shares and shares of four; 128-wide tiles, 3 heads of 100,
    // 54 x 867 x 4, 20 pairs per resident workgroup: 251 and 261, 16 / 4 of 72, 62 x 792 x 2, 12 pairs: 476 and 521; 64-wide, 6 of 48, 34 x 49 x 32,
    // 12 pairs: 98 and 104), as with one workgroup per CU (n > 64, 12 of 100, 100 x 128 x 10, 711 and 756).  Whole rows share no lines: no difference.
    const bool in_step = NARROW && TM == 2 && units >= (D == 128 ? 22 : 13) * most;
    // (a grid dimension holds fewer than 2^32 threads, and a workgroup has up to 256 here; from 67 million pairs on the shares are larger)
    const uint32_t grid = (uint32_t)(in_step ? (units / 4 < 0xffffff ? units / 4 : 0xffffff) & ~(int64_t)7 : units < most ? units : most);
    if (smem > 64 * 1024) {
        const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(mfma_bwd_resident_kernel<D, TM, MODE, NARROW, ROPE>), (int)smem);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((mfma_bwd_resident_kernel<D, TM, MODE, NARROW, ROPE>), dim3(grid), dim3(128 * sp.tiles), smem, s, bp, sp, (uint32_t)units);
    return hipGetLastError();
}

template <int D, bool NARROW, bool ROPE>
hipError_t launch_resident(const BwdParams& bp, hipStream_t s) {
    const int mode = bp.hop.G == 1 ? kOne : bp.hop.vin_heads == bp.hop.Hq ? kHeads : kGroup;
    if (bp.hop.n <= 2 * kTile)
        return mode == kOne ? launch_resident<D, 2, kOne, NARROW, ROPE>(bp, s) : mode == kHeads ? launch_resident<D, 2, kHeads, NARROW, ROPE>(bp, s)
             : launch_resident<D, 2, kGroup, NARROW, ROPE>(bp, s);
    return mode == kOne ? launch_resident<D, 4, kOne, NARROW, ROPE>(bp, s) : mode == kHeads ? launch_resident<D, 4, kHeads, NARROW, ROPE>(bp, s)
         : launch_resident<D, 4, kGroup, NARROW, ROPE>(bp, s);
}

}  // namespace

hipError_t launch_mfma_backward_resident(const BwdParams& bp, hipStream_t s) {
    const int D = bp.hop.D;
    if (bp.hop.rope) return D == 128 ? launch_resident<128, false, true>(bp, s) : D == 64 ? launch_resident<64, false, true>(bp, s)
                          : D > 64 ? launch_resident<128, true, true>(bp, s) : launch_resident<64, true, true>(bp, s);
    return D == 128 ? launch_resident<128, false, false>(bp, s) : D == 64 ? launch_resident<64, false, false>(bp, s)
         : D > 64 ? launch_resident<128, true, false>(bp, s) : launch_resident<64, true, false>(bp, s);
}

}  // namespace ta
