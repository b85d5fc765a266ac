// Device code of the bf16 scoring pass: the projection, row-norm-squared and
// key-value combination steps of Algorithm 1, for gfx950.  Shared by the stand-alone
// scoring kernel and the fused kernel.
//
// The projection is computed transposed, Y^T = G^T A^T (A = K_i or V_i), with
// mfma_f32_16x16x32_bf16: G^T is the A operand (M = 16 sketch columns), a
// sub-tile of 16 token rows is the B operand (N = 16 tokens).  A wave works
// through a contiguous range of 32-token tiles in pairs (64 tokens); a tile is
// two sub-tiles.  In a sub-tile lane L owns token L%16 and, at MFMA step s
// (0..3), the 16 bytes holding d in [s*32 + (L/16)*8, +8): the four lanes of a
// token read 64 contiguous bytes per load instruction and the wave reads whole
// 256-byte rows over the four steps, which the memory system serves as well as
// a fully coalesced stream.  The accumulator of lane L holds sketch coordinates
// cb*16 + 4*(L/16) + {0..3} of token L%16, so the row-norm squared is a sum in
// the lane plus exchanges between the four 16-lane rows, done with the gfx950
// lane-swap instructions (no LDS round trip).  After the exchange every lane of
// a token holds its score; lane row j keeps the score of sub-tile j of the pair,
// so a pair ends with lane L holding the score of token 64*pair + L.  The
// projected rows never leave registers, and scores go to LDS: a global store
// inside the streaming loop costs several percent of the read bandwidth.
#pragma once

#include <type_traits>

#include "curdkv_internal.h"
#include "raw_hist.h"

namespace curdkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) unsigned int words4;

union Chunk {           // 16 bytes of a token row: 8 bf16
    uint4 u;
    bf16x8 v;
};

// How rows are fetched.  STREAM = false: a load instruction asks for 64 bytes of each of 16 rows, in operand layout, and leaves the rows
// in the caches, for a call that reads them again (a gather) or was called right after they were written.  STREAM = true, for calls
// that read more than the caches hold (stream_rows in scores_kernels.hip): whole 128-byte lines, 8 rows an instruction, marked
// non-temporal, which spares the Infinity Cache the filling.  Non-temporal loads of half lines fetch lines twice.  Plain reads of 512 MB and
// 2 GB by 1024 such waves, us: half lines 95.6 and 357, non-temporal 94.8 and 362; whole lines 95.1 and 357, non-temporal 81.8 and 312 (6.9 TB/s).
// The loads of 16 rows come in pairs (a, b) of 128 bytes a row: for a, lanes (tok, q) take 16-byte piece q of row tok (tok < 8) or q + 4 of row tok - 8,
// for b the same of rows 8..15; settle_pair then exchanges between the halves of every 16 lanes, three register moves a word.
// Parts of a streamed scan go through the caches all the same, by ordinary loads of whole lines (kStreamParts, CachedShares): a large one's start, to push out what was written
// just before, and the end of one that gathers many rows afterwards.
constexpr int kStreamNone = 0, kStreamAll = 1, kStreamParts = 2;

template <bool STREAM>
__device__ __forceinline__ int load_row(int tok, int which) { return STREAM ? (tok & 7) + 8 * which : tok; }
template <bool STREAM>
__device__ __forceinline__ int load_piece(int tok, int q, int which) { return STREAM ? q + ((tok >> 3) << 2) : q + 4 * which; }
template <bool STREAM, class W>
__device__ __forceinline__ W fetch(const W* p) {
    if constexpr (STREAM) return __builtin_bit_cast(W, __builtin_nontemporal_load(reinterpret_cast<const words4*>(p)));
    else return *p;
}
// After it lane (tok, q) has pieces q (in a) and q + 4 (in b) of row tok, as without STREAM.
template <class W>
__device__ __forceinline__ void settle_pair(W& a, W& b) {
    words4 x = __builtin_bit_cast(words4, a), y = __builtin_bit_cast(words4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int lo = (int)x[i], hi = (int)y[i];
        x[i] = (unsigned)__builtin_amdgcn_update_dpp(lo, hi, 0x128, 0xF, 0xC, false);   // row_ror:8 into lanes 8..15 of each 16,
        y[i] = (unsigned)__builtin_amdgcn_update_dpp(hi, lo, 0x128, 0xF, 0x3, false);   // and into lanes 0..7
    }
    a = __builtin_bit_cast(W, x);
    b = __builtin_bit_cast(W, y);
}

struct TileRegs {       // one 32-token tile of K and of V as seen by a lane
    Chunk k[2][4];
    Chunk v[2][4];
};

template <int CB>       // CB = padded sketch width / 16
struct SketchRegs {
    bf16x8 g[CB][4];
};

template <int CB>
__device__ __forceinline__ void load_sketch(SketchRegs<CB>& G, const uint4* __restrict__ Gp_head, int lane) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            Chunk c;
            c.u = Gp_head[(cb * 4 + s) * 64 + lane];
            G.g[cb][s] = c.v;
        }
}

// a[32..63] <-> b[0..31]
__device__ __forceinline__ void swap_halves(float& a, float& b) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
// odd 16-lane rows of a <-> even 16-lane rows of b
__device__ __forceinline__ void swap_rows(float& a, float& b) {
    const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// lk, lv: per-lane partial sums of a token held by lanes t, t+16, t+32, t+48.
// Returns (sum of the four lk) * (sum of the four lv) in all four lanes.
__device__ __forceinline__ float combine_rows(float lk, float lv) {
    swap_halves(lk, lv);                 // lk = [lk rows 0,1 | lv rows 0,1], lv = [lk rows 2,3 | lv rows 2,3]
    float x = lk + lv;                   // rows: lk0+lk2, lk1+lk3, lv0+lv2, lv1+lv3
    float y = x;
    swap_rows(x, y);                     // x = rows 0,0,2,2 ; y = rows 1,1,3,3
    float z = x + y;                     // rows: LK, LK, LV, LV
    float w = z;
    swap_halves(z, w);                   // z = LK everywhere, w = LV everywhere
    return z * w;
}

// Scores tiles [t_begin, t_end) of one head; the score of token `row` is written
// to lds_rows[row - row0].  t_begin must be even, and t_end even or equal to
// ceil(n/32): tiles are handled in pairs and a missing second tile is taken to
// lie beyond n.  Returns this lane's sum of the scores it wrote.  Kh, Vh: the
// head's rows, 16 chunks of 16 bytes each.  Token and tile numbers are 32-bit
// (n < 2^31) to keep the address arithmetic out of the register budget.
//
// SRC selects the ablation of the appendix ("Ablation Study"): kSrcKV is the
// method itself (product of key and value scores), kSrcK / kSrcV score from one
// tensor only and never load the other.  PROJ = false drops the sketch: the score
// is the squared norm of the stored row (the four lanes of a token hold 32 of its
// 128 elements each), so no MFMA and no G.
constexpr int kSrcKV = 0, kSrcK = 1, kSrcV = 2;

__device__ __forceinline__ float chunk_sum_sq(const Chunk& c, float acc) {
    const uint32_t w[4] = {c.u.x, c.u.y, c.u.z, c.u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float lo = __uint_as_float(w[i] << 16), hi = __uint_as_float(w[i] & 0xFFFF0000u);
        acc = fmaf(lo, lo, acc);
        acc = fmaf(hi, hi, acc);
    }
    return acc;
}

// Phase of a wave's walk (see scan_tiles): odd multipliers, so that neighbouring heads and
// neighbouring waves of a head start at different offsets.
__device__ __forceinline__ uint32_t scan_phase(int head, int wave_of_head) {
    return (uint32_t)head * 5u + (uint32_t)wave_of_head * 3u;
}

struct CachedTiles { int32_t start_to, end_from; };             // of a wave's walk, in its order: those before start_to and from end_from on

__device__ __forceinline__ CachedTiles cached_tiles(int32_t begin, int32_t end, CachedShares share) {
    const int64_t len = begin < end ? end - begin : 0;
    return {begin + (int32_t)((len * share.start) >> 8), end - (int32_t)((len * share.end) >> 8)};
}

// The walk over tiles [t_begin, t_end) of one wave, shared by the storage types: two tile
// buffers, tiles taken in pairs.
//   load_tile(Tile&, tile, check, how)  issues the loads of one tile; check = std::true_type clamps
//                                   rows to n - 1 (a ragged last tile), std::false_type is for
//                                   tiles known to lie entirely below n: no clamping, no
//                                   predicate, hence no branch, which keeps the steady-state
//                                   loop one basic block so that the compiler's wait counts let
//                                   loads stay in flight; how = std::false_type (kStreamParts, `cached`):
//                                   rows that go through the caches;
//   compute_tile(Tile&, slot)       scores the tile, once per load of it, as first (0) or second (1) of its pair;
//   store_pair(tile, check)         puts the pair's 64 scores away (tile = its first tile).
// t_begin must be even, and t_end even or equal to ceil(n/32): a missing second tile is taken
// to lie beyond n.
template <int MODE, class Tile, class Load, class Compute, class Store>
__device__ __forceinline__ void walk_tiles(int32_t n, int32_t t_begin, int32_t t_end, uint32_t phase, CachedTiles cached,
                                           Load load_tile, Compute compute_tile, Store store_pair) {
    const std::true_type checked, past;
    const std::false_type unchecked, through;
    if (t_begin < t_end) {
        Tile ra, rb;
        const int32_t full = n / kTileTokens;                   // tiles with all 32 rows below n
        // The walk starts at tile t_begin + rot and wraps at t_end; rot follows from the caller's
        // phase.  Heads lie a power of two apart in memory, so waves of different heads that walk
        // from the same offset of their ranges keep asking the same memory channels for different
        // rows; started at different offsets they stream 2-3 % faster (measured, 256 heads of
        // 32768 tokens).  Only ranges of whole pairs of whole tiles are rotated, by whole pairs.
        const int32_t len = t_end - t_begin;
        const int32_t rot = (t_end <= full && !(len & 1) && len >= 8) ? (int32_t)(phase % (uint32_t)(len >> 1)) * 2 : 0;
        auto at = [&](int32_t i) -> int32_t { const int32_t t = i + rot; return t >= t_end ? t - len : t; };
        int32_t t = t_begin;
        // both buffers are always filled (a lone tile is simply loaded twice): a
        // conditional load here would make every wait in the loop below pessimistic
        load_tile(ra, at(t), checked, past);
        load_tile(rb, t + 1 < t_end ? at(t + 1) : at(t), checked, past);
        const int32_t t_steady = t_end < full ? t_end : full;
        auto steady = [&](int32_t until, auto how) {            // until: tiles t .. t+3 of the walk are whole
            for (; t + 4 <= until; t += 2) {
                compute_tile(ra, 0);
                __builtin_amdgcn_sched_barrier(0);
                load_tile(ra, at(t + 2), unchecked, how);
                __builtin_amdgcn_sched_barrier(0);
                compute_tile(rb, 1);
                __builtin_amdgcn_sched_barrier(0);
                load_tile(rb, at(t + 3), unchecked, how);
                store_pair(at(t), unchecked);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto finish = [&](auto how) {                           // last one or two pairs
            for (; t < t_end; t += 2) {
                compute_tile(ra, 0);
                if (t + 2 < t_end) load_tile(ra, at(t + 2), checked, how);
                if (t + 1 < t_end) {
                    compute_tile(rb, 1);
                    if (t + 3 < t_end) load_tile(rb, at(t + 3), checked, how);
                }
                store_pair(at(t), checked);                     // an absent second tile lies beyond n
            }
        };
        if constexpr (MODE == kStreamParts) {                   // (a kernel of its own: the code of both ways costs short scans 3 %)
            steady(cached.start_to < t_steady ? cached.start_to : t_steady, through);
            steady(cached.end_from < t_steady ? cached.end_from : t_steady, past);
            if (cached.end_from < t_end) {
                steady(t_steady, through);
                finish(through);
            } else finish(past);
        } else {
            steady(t_steady, past);
            finish(past);
        }
    }
}

// COUNT: every score is also counted in `hist` (raw_hist_count), those of the first n_sink rows as nothing:
// one LDS atomic per 64 tokens, and the histogram written at the end (scan of 32 heads of 40000 tokens 114.7 us without,
// 116.4 with it, of 8 of 131072 84.0 and 84.8, which saves a pass over the scores).
template <int CB, int SRC = kSrcKV, bool PROJ = true, bool COUNT = false, int MODE = kStreamNone>
__device__ __forceinline__ float scan_tiles(const SketchRegs<CB>& G, const uint4* __restrict__ Kh,
                                            const uint4* __restrict__ Vh, int32_t n, int32_t t_begin,
                                            int32_t t_end, float* lds_rows, int32_t row0, int lane,
                                            uint32_t phase, uint32_t* hist, int32_t n_sink, CachedTiles cached) {
    constexpr bool STREAM = MODE != kStreamNone;
    const int tok = lane & 15, q = lane >> 4;
    float acc_sum = 0.f;
    float pend = 0.f;                                           // this lane's score of the current pair

    auto load_tile = [&](TileRegs& r, int32_t tile, auto check, auto how) {
        constexpr bool kPast = STREAM && decltype(how)::value;
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            size_t off[2];
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                int32_t row = tile * kTileTokens + t2 * 16 + load_row<STREAM>(tok, w);
                if (decltype(check)::value) row = row < n ? row : n - 1;   // ragged tail: reload the last row
                off[w] = (size_t)(uint32_t)row * 16 + load_piece<STREAM>(tok, q, w);
            }
            if (SRC != kSrcV) {
#pragma unroll
                for (int s = 0; s < 4; ++s) r.k[t2][s].u = fetch<kPast>(Kh + off[s & 1] + (s >> 1) * 8);
            }
            if (SRC != kSrcK) {
#pragma unroll
                for (int s = 0; s < 4; ++s) r.v[t2][s].u = fetch<kPast>(Vh + off[s & 1] + (s >> 1) * 8);
            }
        }
    };
    auto compute_tile = [&](TileRegs& r, int slot) {      // slot: 0 = first tile of the pair
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            if constexpr (STREAM) {
#pragma unroll
                for (int s = 0; s < 4; s += 2) {
                    if (SRC != kSrcV) settle_pair(r.k[t2][s], r.k[t2][s + 1]);
                    if (SRC != kSrcK) settle_pair(r.v[t2][s], r.v[t2][s + 1]);
                }
            }
            // a tensor that is not scored contributes 1/4 per lane: four lanes make exactly 1
            float lk = SRC == kSrcV ? 0.25f : 0.f, lv = SRC == kSrcK ? 0.25f : 0.f;
            if (PROJ) {
                f32x4 ak[CB], av[CB];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) { ak[cb] = f32x4{0.f, 0.f, 0.f, 0.f}; av[cb] = f32x4{0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        if (SRC != kSrcV)
                            ak[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(G.g[cb][s], r.k[t2][s].v, ak[cb], 0, 0, 0);
                        if (SRC != kSrcK)
                            av[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(G.g[cb][s], r.v[t2][s].v, av[cb], 0, 0, 0);
                    }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (SRC != kSrcV) lk = fmaf(ak[cb][e], ak[cb][e], lk);
                        if (SRC != kSrcK) lv = fmaf(av[cb][e], av[cb][e], lv);
                    }
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    if (SRC != kSrcV) lk = chunk_sum_sq(r.k[t2][s], lk);
                    if (SRC != kSrcK) lv = chunk_sum_sq(r.v[t2][s], lv);
                }
            }
            const float lkv = combine_rows(lk, lv);
            pend = (q == slot * 2 + t2) ? lkv : pend;
        }
    };
    auto store_pair = [&](int32_t tile, auto check) {           // lane L holds token tile*32 + L
        const int32_t row = tile * kTileTokens + lane;
        if (!decltype(check)::value || row < n) {
            lds_rows[row - row0] = pend;
            if (COUNT) raw_hist_count(hist, pend, row >= n_sink);
            acc_sum += pend;
        }
    };
    walk_tiles<MODE, TileRegs>(n, t_begin, t_end, phase, cached, load_tile, compute_tile, store_pair);
    return acc_sum;
}

// ---- fp32 storage, at most 32 sketch columns, few tokens ---------------------------------------------
// The same walk and the same lane roles as above with mfma_f32_16x16x4f32: lane L holds token
// L%16 and, of every 64-byte stretch of its row, the 16 bytes (four floats) number L/16, so a
// load instruction again asks for 64 contiguous bytes per row.  One MFMA takes one of the four
// floats as the token operand; its sketch operand in lane L is
// G[(4*s + L/16)*4 + e][16*cb + L%16] for step s = 0..7 and float e = 0..3, 32*CB floats per
// lane in registers.  HBM is the bound here (32 columns are 16 flop/B): splitting the products
// over the bf16 matrix units, as the wider sketches do, measured 2 % slower (256 heads of 16384
// tokens, r = 20: 746 us against 729).
struct TileRegsF32 {    // one 32-token tile of K and of V as seen by a lane
    float4 k[2][8];
    float4 v[2][8];
};

template <int CB>
struct SketchF32 {
    float4 g[CB][8];
};

template <int CB, int SRC = kSrcKV, bool PROJ = true, bool COUNT = false>
__device__ __forceinline__ float scan_tiles_f32(const SketchF32<CB>& G, const float4* __restrict__ Kh,
                                                const float4* __restrict__ Vh, int32_t n, int32_t t_begin,
                                                int32_t t_end, float* lds_rows, int32_t row0, int lane,
                                                uint32_t phase, uint32_t* hist, int32_t n_sink) {
    const int tok = lane & 15, q = lane >> 4;
    float acc_sum = 0.f;
    float pend = 0.f;
    auto load_tile = [&](TileRegsF32& r, int32_t tile, auto check, auto) {
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            int32_t row = tile * kTileTokens + t2 * 16 + tok;
            if (decltype(check)::value) row = row < n ? row : n - 1;
            const size_t off = (size_t)(uint32_t)row * 32 + q;          // 32 float4 per row
            const float4* kp = Kh + off;
            const float4* vp = Vh + off;
            if (SRC != kSrcV) {
#pragma unroll
                for (int s = 0; s < 8; ++s) r.k[t2][s] = kp[s * 4];
            }
            if (SRC != kSrcK) {
#pragma unroll
                for (int s = 0; s < 8; ++s) r.v[t2][s] = vp[s * 4];
            }
        }
    };
    auto compute_tile = [&](const TileRegsF32& r, int slot) {
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            float lk = SRC == kSrcV ? 0.25f : 0.f, lv = SRC == kSrcK ? 0.25f : 0.f;
            if (!PROJ) {                        // squared norm of the stored row: 32 of its 128 floats per lane
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    if (SRC != kSrcV) {
                        const float4 x = r.k[t2][s];
                        lk = fmaf(x.x, x.x, lk); lk = fmaf(x.y, x.y, lk); lk = fmaf(x.z, x.z, lk); lk = fmaf(x.w, x.w, lk);
                    }
                    if (SRC != kSrcK) {
                        const float4 x = r.v[t2][s];
                        lv = fmaf(x.x, x.x, lv); lv = fmaf(x.y, x.y, lv); lv = fmaf(x.z, x.z, lv); lv = fmaf(x.w, x.w, lv);
                    }
                }
            }
#pragma unroll
            for (int cb = 0; cb < (PROJ ? CB : 0); ++cb) {
                f32x4 ak = f32x4{0.f, 0.f, 0.f, 0.f}, av = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const float4 g = G.g[cb][s];
                    if (SRC != kSrcV) {
                        const float4 x = r.k[t2][s];
                        ak = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x, x.x, ak, 0, 0, 0);
                        ak = __builtin_amdgcn_mfma_f32_16x16x4f32(g.y, x.y, ak, 0, 0, 0);
                        ak = __builtin_amdgcn_mfma_f32_16x16x4f32(g.z, x.z, ak, 0, 0, 0);
                        ak = __builtin_amdgcn_mfma_f32_16x16x4f32(g.w, x.w, ak, 0, 0, 0);
                    }
                    if (SRC != kSrcK) {
                        const float4 x = r.v[t2][s];
                        av = __builtin_amdgcn_mfma_f32_16x16x4f32(g.x, x.x, av, 0, 0, 0);
                        av = __builtin_amdgcn_mfma_f32_16x16x4f32(g.y, x.y, av, 0, 0, 0);
                        av = __builtin_amdgcn_mfma_f32_16x16x4f32(g.z, x.z, av, 0, 0, 0);
                        av = __builtin_amdgcn_mfma_f32_16x16x4f32(g.w, x.w, av, 0, 0, 0);
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (SRC != kSrcV) lk = fmaf(ak[e], ak[e], lk);
                    if (SRC != kSrcK) lv = fmaf(av[e], av[e], lv);
                }
            }
            const float lkv = combine_rows(lk, lv);
            pend = (q == slot * 2 + t2) ? lkv : pend;
        }
    };
    auto store_pair = [&](int32_t tile, auto check) {
        const int32_t row = tile * kTileTokens + lane;
        if (!decltype(check)::value || row < n) {
            lds_rows[row - row0] = pend;
            if (COUNT) raw_hist_count(hist, pend, row >= n_sink);
            acc_sum += pend;
        }
    };
    walk_tiles<kStreamNone, TileRegsF32>(n, t_begin, t_end, phase, CachedTiles{}, load_tile, compute_tile, store_pair);
    return acc_sum;
}

// ---- few tokens in all, either storage ---------------------------------------------------
// A workgroup takes 16 tokens at a time and its waves share the products: wave w has tensor w / CB
// (where both are scored) and the 16 sketch columns of block w % CB.  With a few thousand tokens per
// call the walks above and below leave most of the chip idle behind serial chains: a wave of scan_tiles_f32
// works through 64 tokens of K and V, 512 fp32 MFMAs of 32 cycles (7 us) at 32 columns; here 32 (0.4 us).
// A wave of scan_tiles loads the whole sketch (16 KB at 64 columns) and 64 rows where one or sixteen are new.
// The products are plain fp32 for fp32 storage at every width.  Scoring, us per call before and after,
// fp32: 1 head of 1024 tokens 17.4 -> 8.5 at r = 20, 23.7 -> 9.6 at r = 64, 34.7 -> 12.0 at r = 128; 8
// heads of 2048 tokens 17.9 -> 12.1, 23.8 -> 16.4, 34.9 -> 21.6; 256 heads of one token 7.9 -> 3.4,
// 15.0 -> 4.2, 23.6 -> 7.1; bf16: 1 head of 1024 tokens 7.9 -> 4.3, 8.5 -> 4.9, 10.3 -> 6.0; 256 heads of one
// token 4.4 -> 2.8, 4.7 -> 3.1, 5.5 -> 3.6.
// first, last: the workgroup's range of 16-token steps; `put(row, score)` is called by the lanes
// 0..15 of wave 0, once for each row below n.  red: LDS, two sets of WAVES x 16 floats, taken in turn so
// that one barrier per step is enough.
template <bool F32> struct FewOperand {             // a lane's quarter of a row, 16 bytes at a time
    static constexpr int kSteps = F32 ? 8 : 4;
    using Word = std::conditional_t<F32, float4, Chunk>;
};

template <bool F32, int CB, int SRC, class Put>
__device__ __forceinline__ void scan_few(const typename FewOperand<F32>::Word* __restrict__ Gh,
                                         const typename FewOperand<F32>::Word* __restrict__ Kh,
                                         const typename FewOperand<F32>::Word* __restrict__ Vh, int32_t n, int32_t first,
                                         int32_t last, float (*red)[(SRC == kSrcKV ? 2 : 1) * CB][16], Put put) {
    constexpr int kSteps = FewOperand<F32>::kSteps;             // a row is 4 * kSteps words
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tok = lane & 15, q = lane >> 4;
    const int cb = wave % CB;
    const auto* src = SRC == kSrcK || (SRC == kSrcKV && wave < CB) ? Kh : Vh;
    typename FewOperand<F32>::Word x[kSteps], g[kSteps];
    auto load = [&](int32_t step) {
        int32_t row = step * 16 + tok;
        row = row < n ? row : n - 1;                            // rows past the end reload the last one
        const auto* p = src + (size_t)(uint32_t)row * (4 * kSteps) + q;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) x[s] = p[s * 4];
    };
    if (first < last) load(first);
#pragma unroll
    for (int s = 0; s < kSteps; ++s) g[s] = Gh[(cb * kSteps + s) * 64 + lane];
    for (int32_t t = first; t < last; ++t) {
        f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            if constexpr (F32) {
                a = __builtin_amdgcn_mfma_f32_16x16x4f32(g[s].x, x[s].x, a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x4f32(g[s].y, x[s].y, a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x4f32(g[s].z, x[s].z, a, 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x4f32(g[s].w, x[s].w, a, 0, 0, 0);
            } else {
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g[s].v, x[s].v, a, 0, 0, 0);
            }
        }
        if (t + 1 < last) load(t + 1);      // (sent out ahead of the products: slower, the barrier waits for loads as well)
        float l = a[0] * a[0];
#pragma unroll
        for (int e = 1; e < 4; ++e) l = fmaf(a[e], a[e], l);
        float m = l;
        swap_rows(l, m);                                        // l = rows 0,0,2,2; m = rows 1,1,3,3
        l += m;
        m = l;
        swap_halves(l, m);                                      // l = rows 0,1 (twice), m = rows 2,3
        l += m;
        auto& out = red[(t - first) & 1];
        if (lane < 16) out[wave][lane] = l;
        __syncthreads();
        if (wave == 0 && lane < 16) {
            float score = 1.f;
#pragma unroll
            for (int tensor = 0; tensor < (SRC == kSrcKV ? 2 : 1); ++tensor) {
                float sum = out[tensor * CB][lane];
#pragma unroll
                for (int c = 1; c < CB; ++c) sum += out[tensor * CB + c][lane];
                score *= sum;
            }
            if (t * 16 + lane < n) put(t * 16 + lane, score);
        }
    }
}

// ---- fp32 storage, many tokens or more than 32 sketch columns -------------------------------------------
// Lane roles as above; the products go through the bf16 matrix units.  A float is split into three bf16 numbers,
// x = x1 + x2 + x3 (rounded to nearest each time: 8 significant bits and a sign per part
// hold 24 bits; exact from 2^-110 up, below which the third part loses bits as a subnormal), the sketch likewise,
// and x*g is taken as the six products whose size is at least 2^-18 of it:
//     x3*g1 + x1*g3 + x2*g2  +  x1*g2 + x2*g1  +  x1*g1,
// smallest first, accumulated in fp32.  What is left out (x2*g3, x3*g2, x3*g3) is at most 2^-24 of |x*g|, the
// rounding of one fp32 product (|x2| <= 2^-8 and |x3| <= 2^-17 for x in [1, 2)), and 2^-27 at root mean square; a
// product of bf16 numbers is exact: the matrix unit rounds once per 32 terms instead of once per 4.  bf16 has the
// exponents of a float, so rows and sketches of any range need no scaling: the parts of two fp16 numbers with a scale per row and per
// sketch took half the matrix time, but hold 22 to 23 bits, and fewer of a sketch's smaller rows: with 40 channels 2^12 to 2^14 times
// the others and their sketch rows as much smaller, the scores erred by up to 1.2e-5.
// A float whose first part is infinite turns its row into NaN here; rescore_row then does such
// a row again in plain fp32.
//
// The squares of a lane's four columns of every block have a sum each; these are added in double, and the lanes' once for the 64 tokens
// of a group.  Error of a score against 64 bits, normal rows, root mean square (largest): r = 33 5.6e-8 (2.5e-7), r = 64 4.5e-8
// (1.9e-7), r = 128 4.0e-8 (1.6e-7), and the same whatever the channels' sizes are; with one chain of fp32 additions 8.2e-8 (3.7e-7), 8.0e-8 (3.7e-7), 8.7e-8 (3.5e-7).
//
// Why: 4*d*r flop per 1024 bytes of a token's K and V rows made the fp32 matrix units the bound
// from r = 64 on; six bf16 products take 6/16 of their time.  256 heads of 16384
// tokens: r = 64 1148 -> 840 us (HBM alone: 720), r = 128 2146 -> 1310 us (the bf16 units are busy
// two thirds of the time).  The sums in double cost nothing once per group; once per 16 tokens, 0.5 us each (3 heads of 6000 tokens, r = 128, 36.9 us
// against 34.9).
//
// The token operand of MFMA step s (0..3) in lane L are the floats of stretches 2s and 2s + 1,
// d = (2s + e/4)*16 + (L/16)*4 + e%4 for e = 0..7, the sketch operand G[d][16*cb + L%16]: two
// neighbouring float4 of the packed sketch.  The sketch's parts live in LDS
// ([cb][s][part][lane], 12 KB per 16 columns) and are read once per 16 tokens of K and V.
union Parts {           // eight floats as three bf16 operands, largest first
    bf16x8 p[3];
    uint32_t w[3][4];
};

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// two floats rounded to bf16 (nearest even), packed
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}

__device__ __forceinline__ Parts split_bf16(const float4& a, const float4& b) {
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    Parts r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float lo = x[2 * e], hi = x[2 * e + 1];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const uint32_t h = pack_bf16(lo, hi);
            r.w[j][e] = h;
            // exact: at most 16 bits remain after the first part, at most 8 after the second
            lo -= __uint_as_float(h << 16);
            hi -= __uint_as_float(h & 0xFFFF0000u);
        }
    }
    return r;
}

template <int CB> constexpr int kSketchF32Chunks = CB * 4 * 3 * 64;     // 16-byte words in LDS

// The whole workgroup splits the head's packed sketch ([cb][step 0..7][lane] float4) into LDS.
template <int CB, int THREADS>
__device__ __forceinline__ void split_sketch_to_lds(bf16x8* gs, const float4* __restrict__ Gh) {
    for (int i = threadIdx.x; i < CB * 4 * 64; i += THREADS) {          // i = (cb*4 + s)*64 + lane
        const int l = i & 63, cs = i >> 6;
        const Parts p = split_bf16(Gh[cs * 128 + l], Gh[cs * 128 + 64 + l]);
#pragma unroll
        for (int j = 0; j < 3; ++j) gs[(cs * 3 + j) * 64 + l] = p.p[j];
    }
    __syncthreads();
}

// One row's squared projected norm in plain fp32, all lanes of a wave on the row's columns.
template <int CB>
__device__ float rescore_row(const bf16x8* gs, const float* __restrict__ row, int lane) {
    float l = 0.f;
    for (int c = lane; c < 16 * CB; c += 64) {
        float y = 0.f;
        for (int d = 0; d < kHeadDim; ++d) {
            const int at = ((c >> 4) * 4 + (d >> 5)) * 3 * 64 + ((d >> 2) & 3) * 16 + (c & 15);
            const int e = ((d >> 4) & 1) * 4 + (d & 3);
            const float g = ((float)gs[at + 128][e] + (float)gs[at + 64][e]) + (float)gs[at][e];   // exact
            y = fmaf(row[d], g, y);
        }
        l = fmaf(y, y, l);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) l += __shfl_xor(l, off, 64);
    return l;
}

// x[q]: a lane's share of the sum of token q*16 + t, t = lane % 16, whose other shares are in lanes t, t+16, t+32, t+48.  Returns
// in lane q*16 + t the sum of that token.
__device__ __forceinline__ double sum_group(const double (&x)[4]) {
    auto swap = [](auto swap_word, double& a, double& b) {
        float al = __int_as_float(__double2loint(a)), ah = __int_as_float(__double2hiint(a));
        float bl = __int_as_float(__double2loint(b)), bh = __int_as_float(__double2hiint(b));
        swap_word(al, bl);
        swap_word(ah, bh);
        a = __hiloint2double(__float_as_int(ah), __float_as_int(al));
        b = __hiloint2double(__float_as_int(bh), __float_as_int(bl));
    };
    double a = x[0], b = x[1], c = x[2], d = x[3];
    swap(swap_halves, a, c);             // a = [x0 rows 0,1 | x2 rows 0,1], c = [x0 rows 2,3 | x2 rows 2,3]
    swap(swap_halves, b, d);             // x1, x3 likewise
    a += c;                              // rows: x0's 0+2, x0's 1+3, x2's 0+2, x2's 1+3
    b += d;
    swap(swap_rows, a, b);               // a = rows x0's, x1's, x2's, x3's 0+2 ; b = their 1+3
    return a + b;
}

struct TileF32 {        // 16 tokens of K and of V as seen by a lane
    float4 k[8];
    float4 v[8];
};

// Scores tiles [t_begin, t_end) (32 tokens each, as elsewhere) of one head, 64 tokens at a time;
// t_begin must be even, and t_end even or equal to ceil(n/32).  16 tokens are split into parts,
// then the loads of the next 16 go out into the registers just freed and stay in flight while
// the matrix units work on the parts: one buffer of 64 registers and 96 of parts, so that two
// waves share a SIMD and one's splitting runs beside the other's products.  (One wave of two
// 32-token buffers per SIMD took turns at the two: 950 us at r = 64, 1460 at r = 128.  Two chains
// of products per 16 columns and wave, K's and V's, are enough: four measured 3 to 5 % slower.)
template <int CB, int SRC = kSrcKV, bool COUNT = false, bool STREAM = false>
__device__ __forceinline__ float scan_tiles_f32_split(const bf16x8* gs, const float4* __restrict__ Kh,
                                                const float4* __restrict__ Vh,
                                                int32_t n, int32_t t_begin, int32_t t_end, float* lds_rows,
                                                int32_t row0, int lane, uint32_t phase, uint32_t* hist,
                                                int32_t n_sink, CachedTiles cached) {
    const int tok = lane & 15, q = lane >> 4;
    const int32_t groups = (t_end - t_begin + 1) >> 1;          // of 64 tokens
    if (groups <= 0) return 0.f;
    float acc_sum = 0.f;
    TileF32 r;
    // rows past the end reload the last one; their scores are dropped
    auto load = [&](int32_t first, auto how) {
        constexpr bool kPast = STREAM && decltype(how)::value;
        size_t off[2];
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            int32_t row = first + load_row<STREAM>(tok, w);
            row = row < n ? row : n - 1;
            off[w] = (size_t)(uint32_t)row * 32 + load_piece<STREAM>(tok, q, w);     // 32 float4 per row
        }
        if (SRC != kSrcV) {
#pragma unroll
            for (int s = 0; s < 8; ++s) r.k[s] = fetch<kPast>(Kh + off[s & 1] + (s >> 1) * 8);
        }
        if (SRC != kSrcK) {
#pragma unroll
            for (int s = 0; s < 8; ++s) r.v[s] = fetch<kPast>(Vh + off[s & 1] + (s >> 1) * 8);
        }
    };
    double tk[4] = {}, tv[4] = {};                             // a lane's share of the norms of the group's tokens, 16 each
    auto step = [&](int part, int32_t next, auto how) {                   // scores the 16 tokens in r, loads those from `next`
        Parts xk[4], xv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (STREAM) {
                if (SRC != kSrcV) settle_pair(r.k[2 * s], r.k[2 * s + 1]);
                if (SRC != kSrcK) settle_pair(r.v[2 * s], r.v[2 * s + 1]);
            }
            if (SRC != kSrcV) xk[s] = split_bf16(r.k[2 * s], r.k[2 * s + 1]);
            if (SRC != kSrcK) xv[s] = split_bf16(r.v[2 * s], r.v[2 * s + 1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        load(next, how);
        __builtin_amdgcn_sched_barrier(0);
        f32x4 qk = f32x4{0.f, 0.f, 0.f, 0.f}, qv = qk;          // squares, a sum each
        // the lane's offset is made opaque, or the compiler lifts the sketch's loads out of the walk
        int gl = lane;
        asm volatile("" : "+v"(gl));
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            f32x4 ak = f32x4{0.f, 0.f, 0.f, 0.f}, av = f32x4{0.f, 0.f, 0.f, 0.f};
            bf16x8 g[4][3];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < 3; ++j) g[s][j] = gs[((cb * 4 + s) * 3 + j) * 64 + gl];
            auto mac = [&](int s, int jg, int jx) {
                if (SRC != kSrcV) ak = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g[s][jg], xk[s].p[jx], ak, 0, 0, 0);
                if (SRC != kSrcK) av = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g[s][jg], xv[s].p[jx], av, 0, 0, 0);
            };
#pragma unroll
            for (int s = 0; s < 4; ++s) { mac(s, 0, 2); mac(s, 2, 0); mac(s, 1, 1); }
#pragma unroll
            for (int s = 0; s < 4; ++s) { mac(s, 1, 0); mac(s, 0, 1); }
#pragma unroll
            for (int s = 0; s < 4; ++s) mac(s, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (SRC != kSrcV) qk[e] = fmaf(ak[e], ak[e], qk[e]);
                if (SRC != kSrcK) qv[e] = fmaf(av[e], av[e], qv[e]);
            }
            __builtin_amdgcn_sched_barrier(0);                  // or several blocks' loads pile up in registers
        }
        auto total = [](const f32x4& q) { return ((double)q[0] + (double)q[1]) + ((double)q[2] + (double)q[3]); };
        if (SRC != kSrcV) tk[part] = total(qk);
        if (SRC != kSrcK) tv[part] = total(qv);
    };
    // the walk starts at a rotated group, as in walk_tiles (whole groups only)
    const int32_t rot = (t_begin + 2 * groups) * kTileTokens <= n && groups >= 4 ? (int32_t)(phase % (uint32_t)groups) : 0;
    const int32_t base = t_begin * kTileTokens;
    int32_t g = rot;
    load(base + g * 64, std::bool_constant<STREAM>{});
    int32_t i = 0;
    auto walk = [&](int32_t to, auto how) {                     // groups i .. to-1 of the walk
        for (; i < to; ++i) {
            const int32_t first = base + g * 64;
            g = g + 1 == groups ? 0 : g + 1;
            step(0, first + 16, how);
            step(1, first + 32, how);
            step(2, first + 48, how);
            step(3, i + 1 < groups ? base + g * 64 : first + 48, how);   // (at the end these rows once more, from the L2, unused)
            const double lk = SRC == kSrcV ? 1.0 : sum_group(tk), lv = SRC == kSrcK ? 1.0 : sum_group(tv);
            const float pend = (float)(lk * lv);
            const int32_t row = first + lane;
            if (row < n) {
                lds_rows[row - row0] = pend;
                if (COUNT) raw_hist_count(hist, pend, row >= n_sink);
                acc_sum += pend;
            }
        }
    };
    if constexpr (STREAM) {
        auto group = [&](int32_t tile) { const int32_t to = (tile - t_begin) >> 1; return to < groups ? to : groups; };
        int32_t until = group(cached.start_to);
        const int32_t past_to = group(cached.end_from);
#pragma clang loop unroll(disable)
        for (int part = 0; part < 2; ++part) {                  // as in walk_tiles
            walk(until, std::false_type{});
            walk(past_to, std::true_type{});
            until = groups;
        }
    } else walk(groups, std::false_type{});
    if (__any(acc_sum != acc_sum)) {                            // some row is not a number: do those again
        acc_sum = 0.f;
        for (int32_t j = base; j < base + groups * 64; j += 64) {
            const int32_t row = j + lane;
            float v = row < n ? lds_rows[row - row0] : 0.f;
            for (uint64_t bad = __ballot(v != v); bad; bad &= bad - 1) {
                const int b = __ffsll((unsigned long long)bad) - 1;
                const size_t at = (size_t)(uint32_t)(j + b) * kHeadDim;
                const float lk = SRC == kSrcV ? 1.f : rescore_row<CB>(gs, (const float*)Kh + at, lane);
                const float lv = SRC == kSrcK ? 1.f : rescore_row<CB>(gs, (const float*)Vh + at, lane);
                if (lane == b) {
                    if (COUNT) raw_hist_uncount(hist, v, row >= n_sink);
                    v = lk * lv;
                    if (COUNT) raw_hist_count(hist, v, row >= n_sink);
                }
            }
            if (row < n) {
                lds_rows[row - row0] = v;
                acc_sum += v;
            }
        }
    }
    return acc_sum;
}

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    return x;
}

}  // namespace curdkv
