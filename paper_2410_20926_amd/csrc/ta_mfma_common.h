// Pieces shared by the bf16 MFMA kernels (forward and backward): vector types, the
// bf16 pack, the wave-level LDS ordering point, tile geometry and the host-side launch
// geometry.  Internal to the library.
#pragma once

#include "ta_internal.h"

namespace ta {
namespace mfma {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr int kTile = 32;                                 // rows of one MFMA tile
constexpr float kLog2e = 1.4426950408889634f;

__device__ inline uint32_t pack_bf16x2(float lo, float hi) {      // v_cvt_pk_bf16_f32, round to nearest even
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ inline float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ inline void lds_wave_sync() {
    // LDS operations of one wave complete in issue order; this only stops the compiler
    // from moving shared-memory accesses across the point where lanes exchange data.
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ inline f32x16 mma(const u32x4 a, const u32x4 b, const f32x16 c) {   // 32x32x16 bf16, fp32 accumulate
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Rows of a head that is narrower than the tile (NARROW here and in the kernels: a head width that is a multiple of 4 but not of 8 features, or simply
// narrower than the tile): a row holds only `dbytes` bytes (at least 16, a multiple of 8) and starts on a multiple of 8 bytes.
// What lies outside the row reads as zero, so that the tile's extra features are zero in every operand.
__device__ inline u32x4 row_only(u32x4 a, uint32_t lbyte, uint32_t dbytes) {
    if (lbyte + 8 > dbytes) { a.x = 0u; a.y = 0u; }
    if (lbyte + 16 > dbytes) { a.z = 0u; a.w = 0u; }
    return a;
}
// Whether every row of a tensor is whole 16-byte units on 16-byte boundaries, so that row_only is all there is to do (uniform).
__device__ inline bool whole_units(const char* base, uint32_t pitch, uint32_t dbytes) {
    return (((uint32_t)reinterpret_cast<uintptr_t>(base) | pitch | dbytes) & 15u) == 0u;
}
// One lane's 16-byte chunk (8 features starting at byte `lbyte` of the row at `base + rowoff`) for the row gathers, where
// the lanes of a row are consecutive lanes that hold consecutive chunks of the whole tile row (chunk = lane % 8 or
// lane % 16) and every lane of the wave takes part.  NARROW rows start on a multiple of 8 bytes; strided 8-byte halves ask
// for every cache line twice and reach 3.5 TB/s in a plain streaming kernel on 200-byte rows, 16-byte requests on 16-byte
// boundaries 4.65 TB/s, and a branch per request makes every request wait for the one before.  So a lane asks for the
// aligned 16 bytes that start at or 8 bytes before its chunk (those 8 bytes lie inside the tensor's span: the tensor itself
// starts on a 16-byte boundary), never for bytes past the end of the row (a unit that would pass it is replaced by the
// row's last 16 bytes; rows are at least that long), and a row that starts 8 bytes into an aligned unit takes the second
// half of each chunk from the next lane.
// Two parts, the request and what is done with the bytes when they have come.  In one piece the first row's bytes are waited for before
// the last rows are requested (the compiler shares the registers of the halves that are put together), so that the four tiles of the one-tile
// backward waited for memory five times one after the other, and the two of the two-tile forward twice.  In two parts (32 / 8 heads of 96, 32 x 32 x 32, the
// backward hop along the second axis 338 -> 276 us, forward 122 -> 104; 12 heads of 96, 134 x 57 x 8, forward 196 -> 124; 8 / 2 heads of 96, 4 x 3 x 6 x 5 x 3,
// a backward hop 15.3 -> 11.9).  `mis`: the row starts 8 bytes into an aligned unit.
// PER_LANE: a 64-bit address per lane instead, for a kernel that has no registers left for the uniform part.
template <bool NARROW, bool NT, bool PER_LANE = false>
__device__ inline u32x4 gather_request(const char* base, uint32_t rowoff, uint32_t lbyte, uint32_t dbytes, uint32_t& mis) {
    if constexpr (!NARROW) {
        mis = 0u;
        const u32x4* src = reinterpret_cast<const u32x4*>(base + (rowoff + lbyte));
        return NT ? __builtin_nontemporal_load(src) : *src;
    } else if constexpr (PER_LANE) {
        const char* row = base + rowoff;
        mis = (uint32_t)reinterpret_cast<uintptr_t>(row) & 8u;
        const u32x4* src = reinterpret_cast<const u32x4*>(row + (int32_t)(lbyte + 16 <= mis + dbytes ? lbyte - mis : dbytes - 16));
        return NT ? __builtin_nontemporal_load(src) : *src;
    } else {
        // `base` is uniform: a uniform 16-byte boundary and 32-bit offsets from it, so that no address takes two registers
        const uint32_t over = (uint32_t)(reinterpret_cast<uintptr_t>(base) & 8u), at = rowoff + over;
        mis = at & 8u;
        const u32x4* src = reinterpret_cast<const u32x4*>((base - over) + (lbyte + 16 <= mis + dbytes ? at - mis + lbyte : at + dbytes - 16));
        return NT ? __builtin_nontemporal_load(src) : *src;
    }
}
template <bool NARROW>
__device__ inline u32x4 gather_ready(const u32x4 a, uint32_t mis, uint32_t lbyte, uint32_t dbytes) {
    if constexpr (!NARROW) {
        return a;
    } else {
        // the unit that reaches 8 bytes past the end of the row came as the row's last 16 bytes: what it wanted is the second half
        const bool last = lbyte + 8 == dbytes + (mis ? 8 : 0);
        const uint32_t x = last ? a.z : a.x, y = last ? a.w : a.y;
        const uint32_t nx = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x101, 0xf, 0xf, true);   // the next lane's (row_shl:1 within 16 lanes)
        const uint32_t ny = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, 0x101, 0xf, 0xf, true);
        return row_only(mis ? u32x4{a.z, a.w, nx, ny} : u32x4{x, y, a.z, a.w}, lbyte, dbytes);
    }
}
// gather_request that notes its `mis` as bit `at` of `bits`.
template <bool NARROW, bool NT>
__device__ inline u32x4 gather_noted(const char* base, uint32_t rowoff, uint32_t lbyte, uint32_t dbytes, int at, uint32_t& bits) {
    uint32_t mis;
    const u32x4 v = gather_request<NARROW, NT>(base, rowoff, lbyte, dbytes, mis);
    if constexpr (NARROW) bits |= (mis >> 3) << at;
    return v;
}
// A tensor's requested chunks made ready; `mis` has a bit per request.
template <bool NARROW, int N>
__device__ inline void gather_ready_all(u32x4 (&raw)[N], uint32_t mis, const char* base, uint32_t pitch, uint32_t lbyte, uint32_t dbytes) {
    if constexpr (NARROW) {
        if (whole_units(base, pitch, dbytes)) {
#pragma unroll
            for (int i = 0; i < N; ++i) raw[i] = row_only(raw[i], lbyte, dbytes);
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) raw[i] = gather_ready<NARROW>(raw[i], (mis >> i) & 1u, lbyte, dbytes);
        }
    }
}
// A finished output row leaves its row-major LDS tile (`lds_chunk` = this lane's 16-byte chunk of it, `lbyte` bytes into
// the row).  NARROW: as 8-byte pieces that are contiguous within each store instruction (the lane that holds chunk c
// writes piece c of the row, then piece chunks + c), read from LDS in that order: the two halves of a chunk, 16 bytes
// apart from the next lane's, would leave every cache line half written by either instruction.
template <bool NARROW, int CHUNKS>
__device__ inline void store_row_chunk(char* base, uint32_t rowoff, const char* lds_chunk, uint32_t lbyte, uint32_t dbytes) {
    if constexpr (!NARROW) {
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(lds_chunk), reinterpret_cast<u32x4*>(base + (rowoff + lbyte)));
    } else {
        const uint32_t p0 = lbyte / 2, p1 = 8u * CHUNKS + lbyte / 2;   // byte offsets of the two pieces within the row
        const char* lds_row = lds_chunk - lbyte;
        // (through the cache, so that L2 can join a row's first and last line with the neighbouring heads' parts)
        if (p0 + 8 <= dbytes) *reinterpret_cast<u32x2*>(base + (rowoff + p0)) = *reinterpret_cast<const u32x2*>(lds_row + p0);
        if (p1 + 8 <= dbytes) *reinterpret_cast<u32x2*>(base + (rowoff + p1)) = *reinterpret_cast<const u32x2*>(lds_row + p1);
    }
}
template <bool NARROW>
__device__ inline void store_chunk(char* base, uint32_t rowoff, uint32_t lbyte, uint32_t dbytes, const u32x4 v) {
    if constexpr (!NARROW) {
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(base + (rowoff + lbyte)));
    } else {
        // a whole chunk in one store (on an 8-byte boundary where the row starts on one), the row's last 8 bytes on their own
        // (through the cache: a row's first and last cache line may be shared with the neighbouring heads' rows, and
        // L2 can put the parts together before the line goes to memory)
        char* a = base + (rowoff + lbyte);
        if (lbyte + 16 <= dbytes) *reinterpret_cast<u32x4*>(a) = v;
        else if (lbyte + 8 <= dbytes) *reinterpret_cast<u32x2*>(a) = u32x2{v.x, v.y};
    }
}

// Stores of rows, some of which do not exist, without a branch: a lane that has nothing to store gives kNowhere, which the buffer's bounds
// check drops.  A store under a branch may or may not have been issued, so that a later wait for a load (loads and stores are counted
// together, in order) has to wait until every store before it has been written as well.  `base` is uniform, offsets are below
// 2^32 - 512 (fits_u32).
constexpr uint32_t kNowhere = 0xffffffffu;
__device__ inline __amdgpu_buffer_rsrc_t row_buffer(char* base) { return __builtin_amdgcn_make_buffer_rsrc(base, 0, 0xfffffff0u, 0x00020000); }
// A lane's 16-byte chunk `lbyte` bytes into the row at `rowoff`.  NARROW as in store_chunk: whole chunks in one store, a row's last 8 bytes
// in one of their own, through the cache.
template <bool NARROW>
__device__ inline void buffer_store_chunk(__amdgpu_buffer_rsrc_t to, uint32_t rowoff, bool exists, uint32_t lbyte, uint32_t dbytes, const u32x4 v, bool whole = false) {
    if constexpr (!NARROW) {
        __builtin_amdgcn_raw_buffer_store_b128(v, to, exists ? rowoff + lbyte : kNowhere, 0, 2);
    } else {
        __builtin_amdgcn_raw_buffer_store_b128(v, to, exists && lbyte + 16 <= dbytes ? rowoff + lbyte : kNowhere, 0, 0);
        if (!whole) __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.x, v.y}, to, exists && lbyte + 8 == dbytes ? rowoff + lbyte : kNowhere, 0, 0);
    }
}

// The same from a row-major LDS tile (`lds_chunk` = this lane's chunk in it), as store_row_chunk: rows that are not whole 16-byte units leave as 8-byte
// pieces that are contiguous within each store instruction.
template <bool NARROW, int CHUNKS>
__device__ inline void buffer_store_row_chunk(__amdgpu_buffer_rsrc_t to, uint32_t rowoff, bool exists, const char* lds_chunk, uint32_t lbyte, uint32_t dbytes, bool whole) {
    static_assert(NARROW);
    if (whole) {
        __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4*>(lds_chunk), to, exists && lbyte < dbytes ? rowoff + lbyte : kNowhere, 0, 0);
    } else {
        const uint32_t p0 = lbyte / 2, p1 = 8u * CHUNKS + lbyte / 2;   // byte offsets of the two pieces within the row
        const char* lds_row = lds_chunk - lbyte;
        __builtin_amdgcn_raw_buffer_store_b64(*reinterpret_cast<const u32x2*>(lds_row + p0), to, exists && p0 < dbytes ? rowoff + p0 : kNowhere, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b64(*reinterpret_cast<const u32x2*>(lds_row + p1), to, exists && p1 < dbytes ? rowoff + p1 : kNowhere, 0, 0);
    }
}

// ---- rotary encoding of a lane's 16-byte chunk (Sec. 3.2: per-axis positions) ----------------------
// A chunk is 4 interleaved feature pairs (2p, 2p+1), p = 4 * chunk + e.  rope_rates gives the turn of
// each of the lane's pairs per position step, in revolutions; rope_chunk turns the chunk of a row at
// position `pos` (by the negative angle when INVERSE: the transpose, what a gradient needs).  fp32
// throughout; the hardware sine and cosine take revolutions, reduced to [0, 1) first.
__device__ inline void rope_rates(const HopParams& p, int chunk, float (&rev)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) rev[e] = __builtin_amdgcn_exp2f(p.rope_c0 * (float)(4 * chunk + e) + p.rope_c1);
}
__device__ inline void rope_sincos(float pos, const float (&rev)[4], float (&c)[4], float (&s)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float t = __builtin_amdgcn_fractf(pos * rev[e]);
        s[e] = __builtin_amdgcn_sinf(t);
        c[e] = __builtin_amdgcn_cosf(t);
    }
}
template <bool INVERSE = false>
__device__ inline u32x4 rope_apply(const u32x4 x, const float (&c)[4], const float (&s)[4]) {
    u32x4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float lo = bf16_lo(x[e]), hi = bf16_hi(x[e]);
        const float sn = INVERSE ? -s[e] : s[e];
        y[e] = pack_bf16x2(lo * c[e] - hi * sn, lo * sn + hi * c[e]);
    }
    return y;
}
__device__ inline u32x4 rope_chunk(const u32x4 x, float pos, const float (&rev)[4]) {
    float c[4], s[4];
    rope_sincos(pos, rev, c, s);
    return rope_apply(x, c, s);
}
// The same on 8 fp32 values (4 pairs) in registers, e.g. a gradient row chunk before it is rounded.
template <bool INVERSE>
__device__ inline void rope_apply_f32(float (&y)[8], const float (&c)[4], const float (&s)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float lo = y[2 * e], hi = y[2 * e + 1];
        const float sn = INVERSE ? -s[e] : s[e];
        y[2 * e] = lo * c[e] - hi * sn;
        y[2 * e + 1] = lo * sn + hi * c[e];
    }
}

template <int D>
struct Geo {
    static constexpr int kChunks = D / 8;                 // 16-byte chunks per row
    static constexpr int kRowsPerPass = 64 / kChunks;     // rows one wave-wide load covers
    static constexpr int kPasses = kTile / kRowsPerPass;  // loads per lane per 32-row tile
    static constexpr int kPitch = D * 2 + 16;             // bytes, row-major bf16 transit rows
    static constexpr int kVPitch = D * 4 + 32;            // bytes, one interleaved row pair of V (4 pitches = 32 banks mod 64)
    static constexpr int kKSteps = D / 16;                // MFMA steps over the feature axis
    static constexpr int kDTiles = D / 32;                // 32-column tiles of an output
    static constexpr int kBufBytes = (kTile * kPitch > (kTile / 2) * kVPitch) ? kTile * kPitch : (kTile / 2) * kVPitch;
};

// Writes this lane's 16-byte chunks (rows i * kRowsPerPass + lrow) into a row-major tile.
template <int D>
__device__ inline void stage_rows(char* stg, const u32x4 (&raw)[Geo<D>::kPasses]) {
#pragma unroll
    for (int i = 0; i < Geo<D>::kPasses; ++i)
        *reinterpret_cast<u32x4*>(stg + i * Geo<D>::kRowsPerPass * Geo<D>::kPitch) = raw[i];
}

// Operand whose contraction index is the feature: lane (row r32, half hf) reads 8 features
// per 16-wide MFMA step.  Serves as A (rows = tile rows) or B (columns = tile rows).
template <int D>
__device__ inline void read_natural(const char* oprd, u32x4 (&op)[Geo<D>::kKSteps]) {
#pragma unroll
    for (int s = 0; s < Geo<D>::kKSteps; ++s) op[s] = *reinterpret_cast<const u32x4*>(oprd + s * 32);
}

// Operand whose contraction index is the tile row: for feature tile t and 16-row step s2,
// lane (feature 32 t + lane % 32, half hf) gets rows 16 s2 + 8 u + 4 hf + (0..3), u = 0, 1.
// ds_read_b64_tr_b16 works on groups of 16 lanes: lane L of a group supplies the address
// of 4 consecutive features of row (L / 4), at feature offset 4 (L % 4); lane L receives
// feature L of the group's 16, from the 4 rows.
template <int D>
__device__ inline void read_transposed(const char* trbase, u32x4 (&op)[Geo<D>::kDTiles][2]) {
#pragma unroll
    for (int t = 0; t < Geo<D>::kDTiles; ++t)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const char* a0 = trbase + (16 * s2) * Geo<D>::kPitch + 64 * t;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(a0 + 8 * Geo<D>::kPitch));
            const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
            op[t][s2] = u32x4{l2.x, l2.y, h2.x, h2.y};
        }
}

// 16 accumulator values of one lane (rows 8 (r/4) + 4 hf + r % 4) -> two B operands.
__device__ inline void pack_rows(const float (&x)[16], u32x4 (&op)[2]) {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
        op[s2] = u32x4{pack_bf16x2(x[8 * s2 + 0], x[8 * s2 + 1]), pack_bf16x2(x[8 * s2 + 2], x[8 * s2 + 3]),
                       pack_bf16x2(x[8 * s2 + 4], x[8 * s2 + 5]), pack_bf16x2(x[8 * s2 + 6], x[8 * s2 + 7])};
}

__device__ inline uint32_t range_mask(int lo, int hi) {   // bits [lo, hi), 0 <= lo, hi <= 32
    const uint32_t mh = hi >= 32 ? 0xffffffffu : ((1u << hi) - 1u);
    const uint32_t ml = lo >= 32 ? 0xffffffffu : ((1u << lo) - 1u);
    return mh & ~ml;
}

// Tile rows [lo, hi) visible from query row `row` of a fibre occupying tile rows [flo, fhi):
// the causal triangle and a band of width `window` (0 = none).  The same range, read the
// other way round (rows that see key `row`), is seen_range().
__device__ inline void visible_range(int row, int flo, int fhi, int causal, int window, int& lo, int& hi) {
    lo = flo;
    hi = causal ? row + 1 : fhi;
    if (window > 0) { lo = max(lo, row - window + 1); hi = min(hi, row + window); }
}
__device__ inline void seen_range(int row, int flo, int fhi, int causal, int window, int& lo, int& hi) {
    lo = causal ? row : flo;
    hi = fhi;
    if (window > 0) { lo = max(lo, row - window + 1); hi = min(hi, row + window); }
}

// The caller's bit table of the axis (row a, word j: keys 32 j .. 32 j + 31 visible from query
// position a), all ones when there is none.
// `fibre`: the fibre's number on this axis (used when every fibre has a table of its own).
__device__ inline uint32_t table_word(const HopParams& p, uint32_t fibre, int a, int j) {
    return p.mask ? p.mask[(int64_t)fibre * p.mask_fibre_words + a * p.mask_words + j] : 0xffffffffu;
}
// Its transpose for key position c of an axis of at most 32 positions: bit a = query
// position a sees key c.
__device__ inline uint32_t table_column(const HopParams& p, uint32_t fibre, int c) {
    if (!p.mask) return 0xffffffffu;
    const uint32_t* t = p.mask + (int64_t)fibre * p.mask_fibre_words;
    uint32_t col = 0;
    for (int a = 0; a < p.n; ++a) col |= ((t[a] >> c) & 1u) << a;
    return col;
}

// One key tile of an online softmax.  st: the scores S^T of the tile (lane = query row, 16 of its keys, the other 16
// in lane ^ 32); vis32: the keys of the tile this lane's row may attend (bit = key); sl2 = scale * log2(e) > 0.  Updates
// the running maximum m (log2 domain) and sum l, returns the un-normalised weights, rounded to bf16, as B operands, and
// the factor `corr` by which everything accumulated before this tile has to be multiplied.
// The maximum is taken over the raw scores and scaled once, and the scale goes into the exponent's multiply-add; a tile
// that every row of the wave sees completely (inside the causal triangle, no band, table or padding) skips the masking:
// the kernels that walk many tiles spend a good part of their time in this vector arithmetic.
__device__ inline void online_softmax_tile(const f32x16& st, uint32_t vis32, int hf, float sl2, float& m, float& l,
                                           u32x4 (&pop)[2], float& corr) {
    float e[16], tmax = -INFINITY;
    if (__all(vis32 == 0xffffffffu)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) { e[r] = st[r]; tmax = fmaxf(tmax, e[r]); }
    } else {
        const uint32_t vis = vis32 >> (4 * hf);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const bool ok = (vis >> (8 * (r / 4) + (r % 4))) & 1u;
            e[r] = ok ? st[r] : -INFINITY;
            tmax = fmaxf(tmax, e[r]);
        }
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
    if (tmax != -INFINITY) tmax *= sl2;
    const float mnew = fmaxf(m, tmax);
    const float msafe = mnew == -INFINITY ? 0.f : mnew;
    corr = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - msafe);
    m = mnew;
    float psum = 0.f;
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
        uint32_t wds[4];
#pragma unroll
        for (int jp = 0; jp < 4; ++jp) {
            const int r = 8 * s2 + 2 * jp;
            const uint32_t pk = pack_bf16x2(__builtin_amdgcn_exp2f(fmaf(e[r], sl2, -msafe)), __builtin_amdgcn_exp2f(fmaf(e[r + 1], sl2, -msafe)));
            psum += bf16_lo(pk) + bf16_hi(pk);            // sum of the ROUNDED weights
            wds[jp] = pk;
        }
        pop[s2] = u32x4{wds[0], wds[1], wds[2], wds[3]};
    }
    psum += __shfl_xor(psum, 32);
    l = l * corr + psum;
}

// Workgroup numbering of the NARROW instantiations.  Rows that are not whole 64-byte pieces share their first and last
// piece with the neighbouring heads' rows.  Workgroup ids go round the 8 XCDs, so with the plain numbering (head block
// = blockIdx.x, fastest) neighbouring heads are written from different L2s and every shared piece reaches memory as two
// partial writes.  Here each XCD takes runs of 2^run_log2 neighbours in the (blockIdx.y, blockIdx.x) sequence: neighbouring
// head blocks follow each other on one XCD, and their rows, stored through the cache, leave its L2 as whole lines, while the eight XCDs
// stay on neighbouring tokens.  Runs of about 128 rows' heads (one, run, and one run per XCD; 32 x 32 x 32, second axis, us): 32 heads of 96, backward 479,
// 385, 417, of 40 267, 179, 178; 32 / 8 heads of 96 287, 271, 296; 32 heads of 100, forward 173, 161, 172; 4 heads of 40, 64 x 24 x 50 x 2, backward 159, 95, 97.
// The end of the grid, less than eight runs, goes in eight shorter ones, and up to seven workgroups as they come (before, a grid that was no
// multiple of eight lost the order altogether: 12 heads of 100, 30 x 20 x 20 x 4, 261 and 220).
__device__ inline uint32_t xcd_order(uint32_t lin, uint32_t total, uint32_t run_log2) {
    const uint32_t base = lin >> (run_log2 + 3u) << (run_log2 + 3u), l = lin - base;
    if (total - base >= 8u << run_log2) return base + ((l & 7u) << run_log2) + (l >> 3);
    const uint32_t run = (total - base) >> 3;             // the last block: shorter runs, and up to seven workgroups as they come
    return l < 8u * run ? base + (l & 7u) * run + (l >> 3) : lin;
}
constexpr uint32_t kLongestRun = 28;                      // run_log2 of one run per XCD
constexpr uint32_t kAsTheyCome = 31;                      // no order
// (FEW: run_log2 may be kAsTheyCome)
template <bool NARROW, bool FEW = false>
__device__ inline void workgroup_xy(uint32_t& bx, uint32_t& by, uint32_t run_log2 = kLongestRun) {
    bx = blockIdx.x; by = blockIdx.y;
    if constexpr (NARROW) {
        if (FEW && run_log2 == kAsTheyCome) return;
        const uint32_t gx = gridDim.x;
        const uint32_t seq = xcd_order(blockIdx.x + gx * blockIdx.y, gx * gridDim.y, run_log2);
        bx = seq % gx;
        by = seq / gx;
    }
}
// run_log2 for workgroups of `heads` heads each: 128 rows that are neighbours.
inline uint32_t narrow_run_log2(int heads) {
    uint32_t r = 7;
    for (; heads > 1 && r > 4; heads /= 2) --r;
    return r;
}
// The same for kernels with a form for few workgroups: such a call is as long as one workgroup, which the order's divisions come first in (300 drawn calls of up to 8 MB: 0.985 of
// the time up to 180 workgroups, of groups 0.98).  From there to 252 the order is worth as much: taken as they come, a hop's workgroups find the last hop's output in another XCD's
// L2 (0.998; 12 heads of 36, 16 x 27 x 5, 204 to 240 workgroups, 15.2 -> 16.6 us), and from 256 on more (1.005).
inline uint32_t narrow_run_log2(int heads, const dim3& grid) {
    return (uint64_t)grid.x * grid.y * grid.z < 192 ? kAsTheyCome : narrow_run_log2(heads);
}

// Launch geometry computed on the host.
struct TileParams {
    int32_t fpt;          // fibres per 32-row tile (n <= 32), else 1
    int32_t qtiles;       // query tiles per fibre: 1 (n <= 32) or 2
    uint32_t tiles;       // units per (batch, head)
    uint32_t tiles_lo;    // gridDim.y; gridDim.z = B * ceil(tiles / tiles_lo)
    uint32_t tiles_hi;
    uint32_t q_row, k_row, v_row, o_row;   // token pitch of each tensor in BYTES
    float inv_n;          // 1 / n
    uint32_t run_log2;    // narrow rows: see xcd_order
};

// Fills tp for an axis of length p.n walked in `key_tiles` 32-key tiles; false when the
// grid would not fit.
inline bool make_tile_params(const HopParams& p, int key_tiles, TileParams* tp) {
    tp->fpt = key_tiles == 1 ? kTile / p.n : 1;
    tp->qtiles = key_tiles == 1 ? 1 : (p.n + kTile - 1) / kTile;
    const int64_t tiles = key_tiles == 1 ? (p.fibres + tp->fpt - 1) / tp->fpt : p.fibres * tp->qtiles;
    if (tiles <= 0 || tiles > 0x7fffffffLL) return false;
    tp->tiles = (uint32_t)tiles;
    tp->tiles_lo = (uint32_t)(tiles < 32768 ? tiles : 32768);
    tp->tiles_hi = (uint32_t)((tiles + tp->tiles_lo - 1) / tp->tiles_lo);
    if ((int64_t)p.B * tp->tiles_hi > 65535) return false;
    tp->q_row = (uint32_t)(p.q.st * 2);
    tp->k_row = (uint32_t)(p.k.st * 2);
    tp->v_row = (uint32_t)(p.vin.st * 2);
    tp->o_row = (uint32_t)(p.o.st * 2);
    tp->inv_n = 1.0f / (float)p.n;
    tp->run_log2 = kLongestRun;
    return true;
}

// Largest byte offset inside one (batch, head) slice must fit 32 bits.
inline bool fits_u32(const Tensor& t, int64_t N) { return (N - 1) * t.st * 2 + 512 < (int64_t)0xffffffffLL; }

}  // namespace mfma
}  // namespace ta
