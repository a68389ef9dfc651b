// Pieces shared by the bf16 MFMA backward kernels: output tiles (transposition, sums, stores) and the visibility of a
// 32 x 32 block of a long axis.  Internal to the library.
#pragma once

#include "ta_mfma_common.h"

namespace ta {
namespace mfma {

template <int D>
struct BGeo : Geo<D> {
    static constexpr int kBuf = kTile * Geo<D>::kPitch;   // one row-major bf16 tile; also 32 rows x 64 fp32 (+pad) for D = 128
    static constexpr int kFPitch = 64 * 4 + 16;           // bytes, fp32 half-tile rows (64 columns)
    static constexpr int kBufBytes = (kBuf > kTile * kFPitch) ? kBuf : kTile * kFPitch;
    static constexpr int kStats = 3 * kTile * 4;          // row max (log2 domain), 1/rowsum, delta
    static constexpr int kWaveBytes = kBufBytes + kStats + kTile * 16;
    static constexpr int kRedBytes = Geo<D>::kDTiles * 16 * 64 * 4;   // one fp32 accumulator set, lane-major
};

// The epilogue's lane -> (row, 16-byte chunk) mapping: pass i of feature half `half` covers
// row 8 i + lane / 8, chunk lane % 8 of the half (8 lanes x 16 B = 128 contiguous bytes).
template <int D>
__device__ inline uint32_t tile_out_offset(const u32x4* rowoff, int which, int half, int i, int lane) {
    const u32x4 off4 = rowoff[8 * i + (lane >> 3)];
    return (which == 0 ? off4.x : which == 1 ? off4.y : off4.z) + (half * 64 + (lane & 7) * 8) * 2;
}

// Requests the current contents of an output tile (for accumulate = 1) long before the
// epilogue needs them, in the epilogue's mapping.
// NARROW (here and below): rows hold only `dbytes` bytes and are 8-byte aligned; see gather_request.
template <int D, bool NARROW = false>
__device__ inline void prefetch_tile(u32x4 (&old)[Geo<D>::kDTiles * 2], const u32x4* rowoff, int which, const char* gbase, int lane,
                                     uint32_t dbytes = 0) {
#pragma unroll
    for (int half = 0; half < Geo<D>::kDTiles / 2; ++half)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (NARROW) {
                // a chunk that would pass the end of the row: the row's last 16 bytes (store_tile takes its half)
                const uint32_t fbyte = (uint32_t)(half * 64 + (lane & 7) * 8) * 2;
                old[half * 4 + i] = *reinterpret_cast<const u32x4*>(gbase + (tile_out_offset<D>(rowoff, which, half, i, lane) - fbyte + min(fbyte, dbytes - 16)));
            } else {
                old[half * 4 + i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(gbase + tile_out_offset<D>(rowoff, which, half, i, lane)));
            }
        }
}

// acc[t][r] holds (row = lane % 32, feature 32 t + 8 (r/4) + 4 hf + r % 4).  Multiplies by
// `mult`, optionally adds the tensor's previous contents (`old`, from prefetch_tile), rounds
// to bf16 and stores the rows with 16-byte stores; the transposition goes through LDS in
// fp32, 64 features at a time.
// No rotation of the stored rows.
struct NoRope {
    static constexpr bool on = false;
    __device__ float pos(int) const { return 0.f; }
    __device__ const HopParams* hop() const { return nullptr; }
};
// The rows are gradients with respect to rotary-encoded rows: tile row r sits at position pos(r) on the
// hop's axis and is turned back (the encoding's transpose) before anything is added to it.
template <typename PosFn>
struct UnRope {
    static constexpr bool on = true;
    const HopParams* p;
    PosFn fn;
    __device__ float pos(int r) const { return fn(r); }
    __device__ const HopParams* hop() const { return p; }
};
template <typename PosFn>
__device__ inline UnRope<PosFn> unrope(const HopParams* p, PosFn fn) { return UnRope<PosFn>{p, fn}; }

// BRANCH: narrow rows that do not exist are left out under a branch.
template <int D, bool NARROW = false, bool BRANCH = !NARROW, typename Enc = NoRope>
__device__ inline void store_tile(const f32x16 (&acc)[Geo<D>::kDTiles], float mult, char* buf, const u32x4* rowoff,
                                  int which, char* gbase, const u32x4 (&old)[Geo<D>::kDTiles * 2], bool add_old, int rows_valid, int lane,
                                  uint32_t dbytes = 0, const Enc enc = Enc{}) {
    using G = BGeo<D>;
    const int r32 = lane & 31, hf = lane >> 5;
#pragma unroll
    for (int half = 0; half < G::kDTiles / 2; ++half) {
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x16& a = acc[2 * half + t2];
                const f32x4 v = {a[4 * q4] * mult, a[4 * q4 + 1] * mult, a[4 * q4 + 2] * mult, a[4 * q4 + 3] * mult};
                *reinterpret_cast<f32x4*>(buf + r32 * G::kFPitch + (32 * t2 + 8 * q4 + 4 * hf) * 4) = v;
            }
        lds_wave_sync();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * i + (lane >> 3), cc = lane & 7;
            const f32x4 x0 = *reinterpret_cast<const f32x4*>(buf + row * G::kFPitch + cc * 32);
            const f32x4 x1 = *reinterpret_cast<const f32x4*>(buf + row * G::kFPitch + cc * 32 + 16);
            // (In front of the branch for whole rows too: the two-tile kernel of four heads has 4 to 8 spilled registers that way, and takes 0.975 of the time nevertheless;
            // 8 / 2 heads of 128, 40 x 4, 19.0 and under the branch 19.6 us.)
            float y[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
            auto value = [&]() {
                if constexpr (Enc::on) {
                    if (enc.hop()->rope) {
                        float rev[4], c[4], sn[4];
                        rope_rates(*enc.hop(), half * 8 + cc, rev);
                        rope_sincos(enc.pos(row), rev, c, sn);
                        rope_apply_f32<true>(y, c, sn);
                    }
                }
                if (add_old) {
                    u32x4 o = old[half * 4 + i];
                    if constexpr (NARROW) {
                        if ((uint32_t)(half * 64 + cc * 8) * 2 + 8 == dbytes) { o.x = o.z; o.y = o.w; }   // the row's last 8 bytes
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) { y[2 * e] += bf16_lo(o[e]); y[2 * e + 1] += bf16_hi(o[e]); }
                }
                return u32x4{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]), pack_bf16x2(y[6], y[7])};
            };
            if constexpr (NARROW && BRANCH) {
                const uint32_t fbyte = (uint32_t)(half * 64 + (lane & 7) * 8) * 2;
                if (row < rows_valid) store_chunk<true>(gbase, tile_out_offset<D>(rowoff, which, half, i, lane) - fbyte, fbyte, dbytes, value());
            } else if constexpr (NARROW) {
                const uint32_t fbyte = (uint32_t)(half * 64 + (lane & 7) * 8) * 2;
                buffer_store_chunk<true>(row_buffer(gbase), tile_out_offset<D>(rowoff, which, half, i, lane) - fbyte, row < rows_valid, fbyte, dbytes, value(), dbytes % 16 == 0);
            } else {
                if (row < rows_valid)
                    __builtin_nontemporal_store(value(), reinterpret_cast<u32x4*>(gbase + tile_out_offset<D>(rowoff, which, half, i, lane)));
            }
        }
        lds_wave_sync();
    }
}

// The same without previous contents to add: the values are rounded to bf16 BEFORE the
// transposition, which then moves half the bytes through LDS (one row-major bf16 tile).
template <int D, bool NARROW = false>
__device__ inline void store_tile_plain(const f32x16 (&acc)[Geo<D>::kDTiles], float mult, char* buf, const u32x4* rowoff,
                                        int which, char* gbase, int rows_valid, int lane, uint32_t dbytes = 0) {
    using G = BGeo<D>;
    const int r32 = lane & 31, hf = lane >> 5;
    const int lrow = lane / G::kChunks, lcol = lane % G::kChunks;
#pragma unroll
    for (int t = 0; t < G::kDTiles; ++t)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            u32x2 v;
            v.x = pack_bf16x2(acc[t][4 * q4] * mult, acc[t][4 * q4 + 1] * mult);
            v.y = pack_bf16x2(acc[t][4 * q4 + 2] * mult, acc[t][4 * q4 + 3] * mult);
            *reinterpret_cast<u32x2*>(buf + r32 * G::kPitch + (32 * t + 8 * q4 + 4 * hf) * 2) = v;
        }
    lds_wave_sync();
#pragma unroll
    for (int i = 0; i < G::kPasses; ++i) {
        const int row = i * G::kRowsPerPass + lrow;
        if constexpr (NARROW) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(buf + row * G::kPitch + lcol * 16);
            buffer_store_chunk<true>(row_buffer(gbase), rowoff[row][which], row < rows_valid, (uint32_t)lcol * 16, dbytes, v, dbytes % 16 == 0);
        } else if (row < rows_valid) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(buf + row * G::kPitch + lcol * 16);
            const u32x4 off4 = rowoff[row];
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(gbase + ((which == 0 ? off4.x : which == 1 ? off4.y : off4.z) + lcol * 16)));
        }
    }
    lds_wave_sync();
}

// Sum of acc over the workgroup's waves in wave order; the total ends in the LAST wave's
// registers.  `red` is a workgroup-shared fp32 area in lane-major layout.
// LONE: with nw = 1 the workgroup's waves have nothing to do with each other.
template <int D, bool LONE = false>
__device__ inline void chain_sum(f32x16 (&acc)[Geo<D>::kDTiles], float* red, int w, int nw, int lane) {
    constexpr int kT = Geo<D>::kDTiles;
    for (int s = 0; s + 1 < nw; ++s) {
        if (w == s) {
#pragma unroll
            for (int t = 0; t < kT; ++t)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    f32x4* cell = reinterpret_cast<f32x4*>(red) + (t * 4 + q4) * 64 + lane;
                    f32x4 v = {acc[t][4 * q4], acc[t][4 * q4 + 1], acc[t][4 * q4 + 2], acc[t][4 * q4 + 3]};
                    if (s > 0) v += *cell;
                    *cell = v;
                }
        }
        __syncthreads();
    }
    if (nw > 1 && w == nw - 1) {
#pragma unroll
        for (int t = 0; t < kT; ++t)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const f32x4 v = *(reinterpret_cast<const f32x4*>(red) + (t * 4 + q4) * 64 + lane);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[t][4 * q4 + e] += v[e];
            }
    }
    if (!LONE || nw > 1) __syncthreads();                 // red may be reused
}

constexpr int kStreamMaxLds = 160 * 1024;              // LDS of one compute unit

struct StreamBwdParams {
    uint32_t q_row, k_row, v_row, o_row;   // token pitch in bytes of Q/dQ, K/dK, the value input and its gradient, dO
    uint32_t fibres_lo, fibres_hi;         // gridDim.y; gridDim.z = B * fibres_hi
    int32_t tiles;                         // ceil(n / 32)
    int32_t parts;                         // the long kernel: workgroups per fibre and key/value head (see parts_of)
};

// Keys 32 c .. 32 c + 31 that query row qr of the fibre may attend (bit = key), and query
// rows 32 a .. 32 a + 31 that may attend key kr (bit = query row).
__device__ inline uint32_t block_vis_keys(const HopParams& p, int64_t fibre, int qr, int c, int nreal) {
    if (qr >= nreal) return 0u;
    int lo, hi;
    visible_range(qr, 0, p.n, p.causal, p.window, lo, hi);
    hi = min(hi, nreal);
    uint32_t v = range_mask(min(max(lo - kTile * c, 0), kTile), min(max(hi - kTile * c, 0), kTile));
    if (p.mask) v &= p.mask[fibre * p.mask_fibre_words + qr * p.mask_words + c];
    return v;
}
__device__ inline uint32_t block_vis_rows(const HopParams& p, int64_t fibre, int kr, int a, int nreal) {
    if (kr >= nreal) return 0u;
    int lo, hi;
    seen_range(kr, 0, p.n, p.causal, p.window, lo, hi);
    hi = min(hi, nreal);
    uint32_t v = range_mask(min(max(lo - kTile * a, 0), kTile), min(max(hi - kTile * a, 0), kTile));
    if (p.mask) {
        const uint32_t* table = p.mask + fibre * p.mask_fibre_words;
        uint32_t col = 0;
#pragma unroll 1
        for (int q = 0; q < kTile; ++q) {                 // rare path: kept rolled, its 32 loads would otherwise claim registers in every kernel
            const int qr = kTile * a + q;
            if (qr < p.n) col |= ((table[qr * p.mask_words + (kr >> 5)] >> (kr & 31)) & 1u) << q;
        }
        v &= col;
    }
    return v;
}

}  // namespace mfma
}  // namespace ta
