// Device code of the per-head selection: the sink, top-k and union steps of
// Algorithm 1, for gfx950.  Shared by the stand-alone selection kernels, the fused
// kernel and the head-wise budget allocation.
//
// A workgroup of THREADS threads handles one (layer, group) with n <= THREADS*KPT.
// Thread t holds the order-preserving 32-bit keys of tokens t, t + THREADS,
// t + 2*THREADS, ... in registers for the whole selection, so every pass over the
// keys is straight-line code with no loads.  The task is to find the key T of the
// (k-s)-th largest candidate and how many keys equal to T are still needed; an
// ordered compaction then lists, in ascending token order, the sinks, every
// candidate above T and the first `need` candidates equal to T, which realises
// "larger score first, then smaller index" exactly.
//
// Finding T, usual case: one histogram over 4096 bins that are a fixed, monotone
// function of the key (bin12: seven exponent bits and five mantissa bits of a score
// below 2, i.e. 32 bins per binade whatever the head's range is), a scan of the
// bins from the top to the bin that holds T, then one more pass over the keys that
// marks every candidate in a higher bin as kept and copies the few candidates
// inside the bin (typically a fraction of a percent of the head) to a list in LDS.
// The remaining 18 key bits are resolved on that list alone, by comparing its keys where they are few, else in three
// 6-bit digits, and the list's members are then marked "above T" or "equal to T".  The keys in
// registers are walked twice in all.
//
// Finding T, general case (the bin holds more keys than the list takes, e.g. a
// head whose scores are all equal, or scores of 2 and above, which all share the
// last bin): most-significant-digit radix select over the keys in registers, 8
// bits at a time, on key - kmin starting at the highest bit in which the head's
// keys differ at all.
//
// The compaction works on bitmaps: one 64-token word per (row, wave) of "above T"
// and of "equal to T" flags; one wave trims the tied flags to the first `need`,
// scans the popcounts into output positions, and then each word's set bits are
// listed.  The indices are collected in an LDS staging array so that the caller
// can write them out, or gather by them, with coalesced accesses.
#pragma once

#include <type_traits>

#include "curdkv_internal.h"

namespace curdkv {

constexpr int kHistRep = 8;                       // general case: replicated bins to thin out LDS atomic collisions
constexpr int kBins12 = 4096;
constexpr int kBinShift = 18;                     // key bits below the bin number (for bins other than the last)

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// What a selection that copies the kept rows itself is given: rows of 16-byte chunks.
struct GatherArgs {
    const u32x4 *K, *V;
    u32x4 *K_out, *V_out;
};

__device__ __forceinline__ uint32_t order_key(float x) {
    x = x + 0.0f;                                 // -0 -> +0
    const uint32_t b = __float_as_uint(x);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Bin of a key: monotone non-decreasing in the key for non-negative scores.  Scores in
// [0, 2) get their exponent and top five mantissa bits; everything from 2 upwards shares
// bin 4095.  Always in [0, 4095], whatever the key.
__device__ __forceinline__ uint32_t bin12(uint32_t key) {
    const uint32_t b = (key & 0x7FFFFFFFu) >> kBinShift;
    return b < (uint32_t)(kBins12 - 1) ? b : (uint32_t)(kBins12 - 1);
}

// The normalisation step of Algorithm 1 applied on the fly: v -> v / (sum of the head), the
// sum being the per-block partial sums added in a fixed order in double; 1/n when the sum
// is 0.  The arithmetic is the one of the stand-alone normalisation kernel.
struct HeadScale {
    float inv, uniform;
    bool zero, on;
    __device__ __forceinline__ float operator()(float v) const {
        return !on ? v : (zero ? uniform : v * inv);
    }
};
// A lane's share of a head's partial sums, one each up to 64; the loads can go out long before head_scale needs them.
__device__ __forceinline__ double head_partial(const float* __restrict__ partial, int blocks) {
    const int lane = threadIdx.x & 63;
    double sum = lane < blocks ? (double)partial[lane] : 0.0;
    if (blocks > 64) {
        static_assert(kMaxBlocksPerHead == 256, "four partial sums a lane");
        float x[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) x[i] = lane + 64 * (i + 1) < blocks ? partial[lane + 64 * (i + 1)] : 0.f;
        sum += (double)x[0] + ((double)x[1] + (double)x[2]);
    }
    return sum;
}
// The sum of a double over the 64 lanes, in every lane: neighbours first, then pairs, and so on, by
// lane exchanges in registers.  All 64 lanes must be there.
__device__ __forceinline__ double wave_total(double x) {
    auto add = [&](auto ctrl) {
        const int lo = __double2loint(x), hi = __double2hiint(x);
        x += __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, decltype(ctrl)::value, 0xF, 0xF, true),
                              __builtin_amdgcn_update_dpp(0, lo, decltype(ctrl)::value, 0xF, 0xF, true));
    };
    using std::integral_constant;
    add(integral_constant<int, 0xB1>{});           // quad_perm 1,0,3,2
    add(integral_constant<int, 0x4E>{});           // quad_perm 2,3,0,1
    add(integral_constant<int, 0x141>{});          // row_half_mirror: the other quad of eight lanes
    add(integral_constant<int, 0x140>{});          // row_mirror: the other half of the row of 16
    {
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
        x = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    }
    {
        const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
        x = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    }
    return x;
}
// What a head's products are multiplied by, tot > 0.  A sum below 2.9e-39, whose reciprocal is no float, must not
// make zeros NaN, which have no place in the order: the largest float instead.
__device__ __forceinline__ float head_reciprocal(double tot) {
    return fminf((float)(1.0 / tot), 3.40282347e38f);
}
// Every wave of every kernel that scales a head adds the same way, so they all agree to the bit.  (One
// after the other, 64 additions that wait for one another take 0.6 us.)
__device__ __forceinline__ HeadScale scale_by(double tot, int64_t n) {
    HeadScale h;
    h.on = true;
    h.zero = !(tot > 0.0);
    h.inv = h.zero ? 0.f : head_reciprocal(tot);
    h.uniform = (float)(1.0 / (double)n);
    return h;
}
__device__ __forceinline__ HeadScale head_scale(double mine, int blocks, int64_t n) {
    if (blocks <= 0) return HeadScale{0.f, 0.f, false, false};
    return scale_by(wave_total(mine), n);
}

// A threshold the caller already knows (the head-wise budget allocation finds one per layer):
// keep every candidate whose key, without its top bit, is above key31, and the first `need`
// candidates equal to it.  key31 = 0xFFFFFFFF: not known, search for it.
struct Threshold {
    uint32_t key31;
    uint32_t need;
};
constexpr uint32_t kNoThreshold = 0xFFFFFFFFu;

// Inclusive prefix sum over the 64 lanes of a wave, in registers: shifts inside the rows of 16 lanes,
// then each row's last value to the rows behind it.  (A chain of __shfl_up goes through the LDS
// unit six times, about 0.3 us when nothing else runs.)
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t x) {
    auto add = [&](auto ctrl, auto rows) {
        x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
    };
    using std::integral_constant;
    add(integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});      // row_shr:1
    add(integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});      // row_shr:2
    add(integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});      // row_shr:4
    add(integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});      // row_shr:8
    add(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});      // row_bcast:15 into rows 1 and 3
    add(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});      // row_bcast:31 into rows 2 and 3
    return x;
}

// What find_bin_from_top reports (in LDS).
struct BinFound {
    uint32_t bin;                                 // the bin in which the running count from the top reaches `want`
    uint32_t rank;                                // the rank wanted inside that bin, counted from its top (>= 1)
    uint32_t count;                               // keys in that bin
};

// Scans BINS counts (a multiple of THREADS) from the top bin downwards and finds the bin in
// which the running count reaches `want` (1 <= want <= total count).  All THREADS threads
// call it; wave_tot is LDS scratch of THREADS/64 words.  Ends with a barrier, after which
// *found may be read.
template <int THREADS, int BINS>
__device__ __forceinline__ void find_bin_from_top(const uint32_t* hist, uint32_t want,
                                                  uint32_t* wave_tot, BinFound* found) {
    constexpr int kPer = BINS / THREADS;           // bins per thread, descending
    static_assert(kPer >= 1 && kPer * THREADS == BINS, "bins must be a multiple of the threads");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t c[kPer], tot = 0;
    if constexpr (kPer % 4 == 0) {                 // (hist is 16-byte aligned)
#pragma unroll
        for (int i = 0; i < kPer; i += 4) {
            const uint4 v = reinterpret_cast<const uint4*>(hist)[(BINS - 4 - tid * kPer - i) / 4];
            c[i] = v.w; c[i + 1] = v.z; c[i + 2] = v.y; c[i + 3] = v.x;
        }
    } else {
#pragma unroll
        for (int i = 0; i < kPer; ++i) c[i] = hist[BINS - 1 - (tid * kPer + i)];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) tot += c[i];
    uint32_t incl = wave_inclusive(tot);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    // the waves' totals by a lane each: one trip to the LDS instead of one per wave
    const uint32_t waves = wave_inclusive(lane < THREADS / 64 ? wave_tot[lane] : 0u);
    const int w = __builtin_amdgcn_readfirstlane(wave);
    const uint32_t before = w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)waves, w - 1) : 0u;
    uint32_t run = before + incl - tot;            // keys in higher bins
    if (run < want && want <= run + tot) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (want <= run + c[i]) {
                found->bin = (uint32_t)(BINS - 1 - (tid * kPer + i));
                found->rank = want - run;
                found->count = c[i];
                break;
            }
            run += c[i];
        }
    }
    __syncthreads();
}

template <int THREADS, int KPT>
struct SelectShared {
    static constexpr int kWaves = THREADS / 64;
    alignas(16) uint32_t hist[kBins12];           // bin12 histogram; later the digit histograms (general case: 256 x kHistRep)
    unsigned long long gmask[KPT * kWaves];       // bitmaps over the tokens, one 64-token word per (row, wave)
    unsigned long long emask[KPT * kWaves];
    uint32_t wpos[KPT * kWaves];                  // output position of a word's first kept token
    uint32_t bin_count[256];                      // general case: bins summed over their replicas
    uint32_t wave_a[kWaves], wave_b[kWaves];
    BinFound found;
    uint32_t digit, want, list_count;
};

// The bin12 histogram of the candidates (tokens s <= j < n) of the keys in registers into
// sm.hist.  All threads call it; sm.hist is complete after the barrier it ends with.
template <int THREADS, int KPT>
__device__ __forceinline__ void build_hist12(const uint32_t (&x)[KPT], int32_t n, int32_t s,
                                             SelectShared<THREADS, KPT>& sm) {
    const int tid = threadIdx.x;
    for (int i = tid; i < kBins12 / 4; i += THREADS) reinterpret_cast<uint4*>(sm.hist)[i] = uint4{0, 0, 0, 0};
    __syncthreads();
    const uint32_t span = (uint32_t)(n - s);
    const uint32_t jt = (uint32_t)(tid - s);       // token - s of row 0, wraps for sinks
#pragma unroll
    for (int it = 0; it < KPT; ++it)
        if (jt + (uint32_t)(it * THREADS) < span) atomicAdd(&sm.hist[bin12(x[it])], 1u);
    __syncthreads();
}

// Writes a bin12 histogram (complete, in LDS) to dst, and its sums per exponent, 32 bins each, to coarse.
template <int THREADS>
__device__ __forceinline__ void hist12_store(const uint32_t* hist, uint32_t* __restrict__ dst, uint32_t* __restrict__ coarse) {
    constexpr int kPer = kBins12 / THREADS;        // neighbouring bins per thread
    static_assert(kPer % 4 == 0 && 32 % kPer == 0, "an exponent's bins lie in neighbouring lanes");
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer / 4; ++i) {
        const uint4 c = reinterpret_cast<const uint4*>(hist)[threadIdx.x * (kPer / 4) + i];
        reinterpret_cast<uint4*>(dst)[threadIdx.x * (kPer / 4) + i] = c;
        sum += (c.x + c.y) + (c.z + c.w);
    }
#pragma unroll
    for (int off = 1; off < 32 / kPer; off *= 2) sum += __shfl_xor(sum, off, 64);
    if (threadIdx.x % (32 / kPer) == 0) coarse[threadIdx.x / (32 / kPer)] = sum;
}

// General case of the threshold search: radix select over the keys in registers.  Fills
// sm.gmask / sm.emask with the "above T" / "equal to T" flags of the candidates and returns
// how many keys equal to T are still to be kept.  x is overwritten.  Ends with a barrier.
template <int THREADS, int KPT>
__device__ __forceinline__ uint32_t threshold_by_radix(uint32_t (&x)[KPT], int32_t n, int32_t s, int32_t m,
                                                       SelectShared<THREADS, KPT>& sm) {
    constexpr int kWaves = THREADS / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t span = (uint32_t)(n - s);
    const uint32_t jt = (uint32_t)(tid - s);
    auto cand = [&](int it) -> bool { return jt + (uint32_t)(it * THREADS) < span; };
    // ---- range [kmin, kmax] of the candidates -----------------------------------
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int it = 0; it < KPT; ++it)
        if (cand(it)) { kmin = x[it] < kmin ? x[it] : kmin; kmax = x[it] > kmax ? x[it] : kmax; }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t a = __shfl_xor(kmin, off, 64), b = __shfl_xor(kmax, off, 64);
        kmin = a < kmin ? a : kmin;
        kmax = b > kmax ? b : kmax;
    }
    if (lane == 0) { sm.wave_a[wave] = kmin; sm.wave_b[wave] = kmax; }
    for (int i = tid; i < 256 * kHistRep; i += THREADS) sm.hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        kmin = sm.wave_a[w] < kmin ? sm.wave_a[w] : kmin;
        kmax = sm.wave_b[w] > kmax ? sm.wave_b[w] : kmax;
    }
    // From here on x = key - kmin for candidates and all-ones for everything else
    // (sinks, tokens beyond n).  Scores are non-negative, so a candidate's x stays
    // below 2^31 and the all-ones value never matches a prefix or the threshold:
    // the passes below need no per-token candidate test.
    constexpr uint32_t kNotCand = 0xFFFFFFFFu;
#pragma unroll
    for (int it = 0; it < KPT; ++it) x[it] = cand(it) ? x[it] - kmin : kNotCand;

    const uint32_t range = kmax - kmin;
    int rem = range ? 32 - __clz(range) : 0;       // bits of x not yet decided
    rem = rem > 31 ? 31 : rem;                     // only reachable with negative scores (not supported)
    uint32_t fixed = 0;                            // decided high part: x >> rem
    uint32_t want = (uint32_t)m;
    uint32_t* myhist = sm.hist + (lane & (kHistRep - 1));
    while (rem > 0) {
        const int w = rem < 8 ? rem : 8;
        const int shift = rem - w;
        const uint32_t dmask = (1u << w) - 1u;
#pragma unroll
        for (int it = 0; it < KPT; ++it)
            if ((x[it] >> rem) == fixed)
                atomicAdd(&myhist[((x[it] >> shift) & dmask) * kHistRep], 1u);
        __syncthreads();
        for (int b = tid; b < 256; b += THREADS) {
            uint32_t c = 0;
#pragma unroll
            for (int r = 0; r < kHistRep; ++r) { c += sm.hist[b * kHistRep + r]; sm.hist[b * kHistRep + r] = 0; }
            sm.bin_count[b] = c;
        }
        __syncthreads();
        if (wave == 0) {
            // lane L looks at bins 255-4L .. 252-4L (descending); find the bin where the
            // count from the top reaches `want`
            uint32_t c[4], tot = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) { c[i] = sm.bin_count[255 - 4 * lane - i]; tot += c[i]; }
            uint32_t incl = wave_inclusive(tot);
            uint32_t run = incl - tot;             // keys in higher bins
            if (run < want && want <= incl) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (want <= run + c[i]) { sm.digit = 255 - 4 * lane - i; sm.want = want - run; break; }
                    run += c[i];
                }
            }
        }
        __syncthreads();
        fixed = (fixed << w) | sm.digit;
        want = sm.want;
        rem = shift;
        // digit/want are next written after two more barriers; the histogram is already clear
    }
    const uint32_t T = fixed;                      // in x space
    // Word w = it*kWaves + wave of a bitmap covers tokens 64w .. 64w+63, so one ballot per
    // row is one word.
    const uint32_t above = kNotCand - 1u - T;      // T < x < all-ones  <=>  x - T - 1 < above
#pragma unroll
    for (int it = 0; it < KPT; ++it) {
        const uint64_t bg = __ballot(x[it] - T - 1u < above), be = __ballot(x[it] == T);
        if (lane == 0) { sm.gmask[it * kWaves + wave] = bg; sm.emask[it * kWaves + wave] = be; }
    }
    __syncthreads();
    return want;                                   // keys equal to T still to be kept (>= 1)
}

// Resolves the 18 key bits below the bin number on a list of (key, token) pairs in LDS:
// pairs[2i] = key, pairs[2i+1] = token of the i-th of `count` candidates, all of bin `bin`
// (< 4095).  `want` = rank of the threshold among them, from the top.  scratch: kListScratch zeroed LDS words,
// digit/want_s LDS words.  Returns
// the threshold as (key & 0x7FFFFFFF) and, through *need, how many keys equal to it are still
// to be kept.  All THREADS threads call it; ends with a barrier.
constexpr uint32_t kListPairs = 128;               // keys up to which every one is compared with every other
constexpr int kListScratch = 64 + (int)kListPairs;

template <int THREADS>
__device__ __forceinline__ uint32_t threshold_on_list(const int32_t* pairs, uint32_t count, uint32_t bin,
                                                      uint32_t want, uint32_t* scratch, uint32_t* digit,
                                                      uint32_t* want_s, uint32_t* need) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (count <= 32u) {
        // a short list (heads up to some 8000 tokens): one wave compares every key with every other, which costs
        // one barrier instead of six (selection of 64 heads of 4096 tokens 6.3 -> 5.9 us; with lists of 50 keys,
        // 32 heads of 20000 tokens, it would be 13.7 -> 14.3)
        if (wave == 0) {
            const uint32_t key = lane < (int)count ? (uint32_t)pairs[2 * lane] & 0x7FFFFFFFu : 0u;
            uint32_t above = 0, equal = 0;
            for (uint32_t i = 0; i < count; i += 8) {          // (lanes past the list hold 0: above nothing)
#pragma unroll
                for (uint32_t u = 0; u < 8; ++u) {
                    const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)key, (int)(i + u));
                    above += other > key ? 1u : 0u;
                    equal += other == key ? 1u : 0u;
                }
            }
            // (equal keys all write the same)
            if (lane < (int)count && above < want && want <= above + equal) { *digit = key; *want_s = want - above; }
        }
        __syncthreads();
        *need = *want_s;
        return *digit;
    }
    if (count <= kListPairs) {
        // all waves compare: a thread has one key and an equal part of the others, which is the same for a wave's threads.
        // Two barriers instead of six: selection of 8 heads of 8192 tokens 7.3 -> 6.9 us, of 112 of 10007 9.5 -> 9.0, the waves'
        // totals in one read (find_bin_from_top) included; up to 256 keys the allotment of 8 heads' budgets took 0.6 us longer than with digits
        const uint32_t places = count <= 64u ? 64u : 128u;      // threads 0 .. places-1 have the first part
        const uint32_t i = (uint32_t)tid & (places - 1u), parts = (uint32_t)THREADS / places;
        const uint32_t per = (count + parts - 1u) / parts;
        const uint32_t j0 = (uint32_t)__builtin_amdgcn_readfirstlane(tid / (int)places) * per;
        const uint32_t j1 = j0 + per < count ? j0 + per : count;
        const uint32_t key = i < count ? (uint32_t)pairs[2 * i] & 0x7FFFFFFFu : 0u;
        uint32_t sums = 0;                         // keys above in the lower half, equal ones in the upper
#pragma unroll 4
        for (uint32_t j = j0; j < j1; ++j) {
            const uint32_t other = (uint32_t)pairs[2 * j] & 0x7FFFFFFFu;
            sums += other > key ? 1u : other == key ? 0x10000u : 0u;
        }
        if (i < count && sums) atomicAdd(&scratch[64 + i], sums);
        __syncthreads();
        if ((uint32_t)tid < count) {               // (equal keys all write the same)
            const uint32_t all = scratch[64 + tid], above = all & 0xFFFFu;
            if (above < want && want <= above + (all >> 16)) { *digit = key; *want_s = want - above; }
        }
        __syncthreads();
        *need = *want_s;
        return *digit;
    }
    uint32_t* hist64 = scratch;
    uint32_t fixed = bin;                          // decided high part of (key & 0x7FFFFFFF): >> rem
    for (int rem = kBinShift; rem > 0; rem -= 6) {
        const int shift = rem - 6;
        for (uint32_t i = tid; i < count; i += THREADS) {
            const uint32_t key = (uint32_t)pairs[2 * i] & 0x7FFFFFFFu;
            if ((key >> rem) == fixed) atomicAdd(&hist64[(key >> shift) & 63u], 1u);
        }
        __syncthreads();
        if (wave == 0) {                           // lane L looks at digit 63 - L
            const uint32_t c = hist64[63 - lane];
            uint32_t incl = wave_inclusive(c);
            if (incl - c < want && want <= incl) { *digit = 63 - lane; *want_s = want - (incl - c); }
            hist64[63 - lane] = 0;
        }
        __syncthreads();
        fixed = (fixed << 6) | *digit;
        want = *want_s;
        // digit/want_s are next written after another barrier
    }
    *need = want;
    return fixed;
}

// x[it]: key of token it*THREADS + tid (any value for tokens >= n).  Writes the k
// selected token indices, ascending, to stage[0..k) (positions >= cap go straight
// to out_global instead).  stage[] is also used as working memory before that.  All
// threads of the workgroup must call it; it ends with a barrier, after which stage[]
// is complete.  0 <= k <= n, 0 <= s <= n, n <= THREADS*KPT < 65536, cap >= 0.
// `given`: the threshold, where the caller knows it (then k - s must be the number of
// candidates above it plus given.need); the search is skipped.
// SHARE: only positions first .. last-1 are listed, at stage[0 .. last-first), which must be room for them.
template <int THREADS, int KPT, bool SHARE = false>
__device__ __forceinline__ void select_core(uint32_t (&x)[KPT], int32_t n, int32_t s, int32_t k,
                                            SelectShared<THREADS, KPT>& sm, int32_t* stage,
                                            int32_t cap, int32_t* out_global,
                                            Threshold given = Threshold{kNoThreshold, 0u}, int32_t first = 0, int32_t last = 0) {
    constexpr int kWaves = THREADS / 64;
    constexpr int kWords = KPT * kWaves;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto put = [&](uint32_t pos, int32_t j) {
        if (SHARE) {
            if (pos - (uint32_t)first < (uint32_t)(last - first)) stage[pos - (uint32_t)first] = j;
        } else if (pos < (uint32_t)cap) stage[pos] = j; else out_global[pos] = j;
    };

    const int32_t sinks = s < k ? s : k;           // budget inside the sink block: tokens 0..k-1
    const int32_t m = k - s;                       // picks among tokens [s, n)
    const uint32_t span = (uint32_t)(n - s);
    if (m <= 0) {
        for (int32_t j = tid; j < sinks; j += THREADS) put(j, j);
        __syncthreads();
        return;
    }
    if ((uint32_t)m >= span) {                     // everything is kept
        for (int32_t j = tid; j < n; j += THREADS) put(j, j);
        __syncthreads();
        return;
    }

    uint32_t need;
    if (given.key31 != kNoThreshold) {
        // ---- the threshold is known: flags straight from the keys -------------------------------
        const uint32_t jt = (uint32_t)(tid - s);
#pragma unroll
        for (int it = 0; it < KPT; ++it) {
            const bool cd = jt + (uint32_t)(it * THREADS) < span;
            const uint32_t k31 = x[it] & 0x7FFFFFFFu;
            const uint64_t bg = __ballot(cd && k31 > given.key31), be = __ballot(cd && k31 == given.key31);
            if (lane == 0) { sm.gmask[it * kWaves + wave] = bg; sm.emask[it * kWaves + wave] = be; }
        }
        need = given.need;
        __syncthreads();
    } else {
    // ---- the bin that holds the threshold ------------------------------------------------
    build_hist12<THREADS, KPT>(x, n, s, sm);
    if (tid == 0) sm.list_count = 0;
    find_bin_from_top<THREADS, kBins12>(sm.hist, (uint32_t)m, sm.wave_a, &sm.found);
    const uint32_t bstar = sm.found.bin;
    const uint32_t in_bin = sm.found.count;        // candidates inside that bin (>= 1)
    const uint32_t rank = sm.found.rank;           // of the threshold inside the bin, from the top
    // the list takes (key, token) pairs in stage[]; the last bin has no fixed width
    if (bstar < (uint32_t)(kBins12 - 1) && (int64_t)in_bin * 2 <= (int64_t)cap) {
        const uint32_t jt = (uint32_t)(tid - s);
        for (int i = tid; i < kWords; i += THREADS) sm.emask[i] = 0ull;
        for (int i = tid; i < kListScratch; i += THREADS) sm.hist[i] = 0;
        // ---- candidates in higher bins are kept; those inside the bin go to the list ---------
#pragma unroll
        for (int it = 0; it < KPT; ++it) {
            const bool cd = jt + (uint32_t)(it * THREADS) < span;
            const uint32_t b = bin12(x[it]);
            const uint64_t bg = __ballot(cd && b > bstar);
            if (lane == 0) sm.gmask[it * kWaves + wave] = bg;
            if (cd && b == bstar) {
                const uint32_t slot = atomicAdd(&sm.list_count, 1u);
                if (slot < in_bin) {               // always true; keeps a write inside the list whatever happens
                    stage[2 * slot] = (int32_t)x[it];
                    stage[2 * slot + 1] = it * THREADS + tid;
                }
            }
        }
        __syncthreads();
        const uint32_t T = threshold_on_list<THREADS>(stage, in_bin, bstar, rank, sm.hist, &sm.digit, &sm.want, &need);
        // ---- the list's members join the bitmaps -------------------------------------------------
        for (uint32_t i = tid; i < in_bin; i += THREADS) {
            const uint32_t key = (uint32_t)stage[2 * i] & 0x7FFFFFFFu;
            const uint32_t j = (uint32_t)stage[2 * i + 1];
            if (key > T) atomicOr(&sm.gmask[j >> 6], 1ull << (j & 63u));
            else if (key == T) atomicOr(&sm.emask[j >> 6], 1ull << (j & 63u));
        }
        __syncthreads();
    } else {
        need = threshold_by_radix<THREADS, KPT>(x, n, s, m, sm);
    }
    }

    // ---- ordered compaction through the bitmaps ------------------------------------------
    if (wave == 0) {
        // lane L owns words L*kPer .. L*kPer+kPer-1.  First scan: tied keys before each word,
        // to cut emask down to the first `need` of them; second scan: output position of
        // each word's first kept token.
        constexpr int kPer = (kWords + 63) / 64;
        uint64_t keep[kPer];
        uint32_t ne = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int w = lane * kPer + i;
            keep[i] = w < kWords ? sm.emask[w] : 0ull;
            ne += (uint32_t)__popcll(keep[i]);
        }
        uint32_t incl = wave_inclusive(ne);
        uint32_t eq_before = incl - ne, nk = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int w = lane * kPer + i;
            uint64_t e = keep[i];
            const uint32_t c = (uint32_t)__popcll(e);
            if (eq_before >= need) e = 0ull;                       // quota already used up
            else if (eq_before + c > need)                         // the word where it runs out
                for (uint32_t drop = eq_before + c - need; drop; --drop) e &= ~(1ull << (63 - __clzll((long long)e)));
            eq_before += c;
            keep[i] = (w < kWords ? sm.gmask[w] : 0ull) | e;
            nk += (uint32_t)__popcll(keep[i]);
        }
        incl = wave_inclusive(nk);
        uint32_t pos = (uint32_t)s + incl - nk;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int w = lane * kPer + i;
            if (w < kWords) { sm.gmask[w] = keep[i]; sm.wpos[w] = pos; }
            pos += (uint32_t)__popcll(keep[i]);
        }
    }
    __syncthreads();                               // the list in stage[] is no longer needed either
    for (int32_t j = tid; j < sinks; j += THREADS) put(j, j);
    // a thread lists the kept tokens of a quarter word (16 tokens), ascending.  Quarter words
    // rather than words bound the walk when the kept tokens are neighbours (sink-like prefixes,
    // recent windows): 60 neighbours in one word cost one thread, and everybody waiting for
    // it, 5 us.
    for (int q = tid; q < kWords * 4; q += THREADS) {
        const int w = q >> 2, part = q & 3;
        const uint64_t word = sm.gmask[w];
        uint32_t mm = (uint32_t)(word >> (16 * part)) & 0xFFFFu;
        uint32_t pos = sm.wpos[w] + (uint32_t)__popcll(word & ((1ull << (16 * part)) - 1ull));
        if (SHARE && (pos >= (uint32_t)last || pos + 16 <= (uint32_t)first)) continue;
        while (mm) {
            const int bit = __ffs(mm) - 1;
            mm &= mm - 1;
            // positions stay below k by construction; the comparison keeps a write inside
            // the group's slice whatever the keys were
            if (pos < (uint32_t)k) put(pos, w * 64 + 16 * part + bit);
            ++pos;
        }
    }
    __syncthreads();
}

}  // namespace curdkv
