// Selection of long heads by several workgroups per (layer, group), for gfx950: the sink, top-k
// and union steps of Algorithm 1 where one workgroup per head (select_kernels.hip) would leave
// most of the chip idle, or would stream a head that does not fit its registers through one
// compute unit.  Three steps, each a barrier for the next:
//   1. histograms of the scores over 4096 bins (exponent and top four mantissa bits), one per
//      workgroup that makes them: the scoring kernel, on the one-call path, while it has the
//      (un-normalised) scores in LDS, or split_hist_kernel from scores in memory;
//   2. split_flag_kernel, workgroup (head, part): every workgroup finds the bin that holds the
//      cut (the same small sums in each: exponents first, then the sixteen bins of one
//      exponent), turns it into a range [lo, hi] of normalised scores and writes one bit per
//      token of its part to two bitmaps, "above hi" and "in the range".  On the one-call
//      path it also normalises the scores;
//   3. split_emit_kernel, workgroup (head, share): reads the head's bitmaps (n/4 bytes), resolves
//      the threshold on the few keys in the range, scans the popcounts into output positions
//      and lists its share of the output rows.  Resolving and scanning are repeated
//      by every workgroup of a head: they are small, and it saves a launch and a trip through
//      memory.
// What is kept and in which order is exactly what select_core (select_device.h) keeps.
//
// Normalising multiplies by one factor and rounds, so it keeps the order of two products or makes
// them equal.  The m-th largest score is therefore the normalised m-th largest product, and
// lies in the normalised range of that product's bin; products of neighbouring bins that round
// onto the range's ends are inside the range too, so that ties between them are
// decided by token number as everywhere.
//
// The range is a sixteenth of a binade: a few hundred to a few thousand tokens of a long head whose scores spread
// over decades, but a tenth or more of one whose scores lie together (rows of like norm).  Step 3 takes up to 4096 keys in
// LDS, up to 20480 in registers, and narrows a fuller range by reading its scores again, a digit per pass.
// Without the registers, us per call: 8 heads of 131072 normal rows, 64 columns, half kept, 361, with them 210 (one
// workgroup per head: 271); 128 columns, a tenth kept, 309 and 147 (208); 64 heads of 65536, 64 columns, half kept, 807 and 739 (750).
//
// (One histogram per head, added up with atomics, took 15 us for 8 heads of 131072 tokens where
// writing and summing one per workgroup takes about 1: atomics of many workgroups on one address
// go through memory one after the other on this chip.)

#include "raw_hist.h"
#include "select_device.h"

namespace curdkv {

constexpr int kSplitThreads = 512;
constexpr int kSplitWaves = kSplitThreads / 64;
constexpr int kSplitPairs = 4096;                  // keys in the range that step 3 resolves in LDS,
constexpr int kSplitList = 20480;                  // and in registers: two workgroups still share a unit's LDS
constexpr int kSplitMinTokens = 24 * 1024;          // one call, at most 32 heads
constexpr int kSplitMinTokensElse = 36 * 1024;      // beyond: one workgroup's registers hold a head up to here
constexpr int kSplitMaxTokens = 131072;            // tokens per head the bitmaps and their scan are laid out for
constexpr int kSplitMaxWords = kSplitMaxTokens / 64;
constexpr int kSplitWordsPerThread = kSplitMaxWords / kSplitThreads;   // 4
constexpr int kSplitShare = 1024;                  // output rows a workgroup of step 3 lists at most, where it also gathers them

struct SplitWorkspace {                            // device pointers into one allocation; nothing survives a call
    uint32_t* hist;                                // [heads][hists][2048], two 16-bit counts to a word
    uint32_t* coarse;                              // [heads][hists][256], per exponent
    unsigned long long* gmask;                     // [heads][words]
    unsigned long long* emask;                     // [heads][words]
    uint2* range;                                  // [heads] keys lo, hi (without the top bit)
    int words, hists;                              // allocated per head
};

static int words_for(int64_t max_tokens) {
    const int64_t t = max_tokens < kSplitMaxTokens ? max_tokens : kSplitMaxTokens;
    return (int)(((t + 63) / 64 + 1) & ~(int64_t)1);
}

// histograms per head: what pick_blocks_per_head (scores_kernels.hip) can ask for; fewer heads, more workgroups each
int split_hists(const curdkv_ctx* ctx) { return ctx->heads <= 32 ? 64 : 32; }

static SplitWorkspace carve(const curdkv_ctx* ctx) {
    SplitWorkspace w;
    const size_t heads = (size_t)ctx->heads;
    w.words = words_for(ctx->cfg.max_tokens);
    w.hists = split_hists(ctx);
    w.hist = reinterpret_cast<uint32_t*>(ctx->d_split_ws);
    w.coarse = w.hist + heads * w.hists * kRawHistWords;
    w.gmask = reinterpret_cast<unsigned long long*>(w.coarse + heads * w.hists * 256);
    w.emask = w.gmask + heads * w.words;
    w.range = reinterpret_cast<uint2*>(w.emask + heads * w.words);
    return w;
}

size_t split_workspace_bytes(const curdkv_ctx* ctx) {
    return (size_t)ctx->heads * ((size_t)split_hists(ctx) * (kRawHistWords + 256) * 4 + (size_t)words_for(ctx->cfg.max_tokens) * 16 + sizeof(uint2));
}

struct SplitArgs {
    SplitWorkspace ws;
    float* scores;
    int32_t n, n_sink;
    const int64_t* offsets;
    const float* partial;
    int scale_blocks, write_scaled;                // as in launch_select
    int part;                                      // tokens per workgroup of step 2, a multiple of 512
    int hists;                                     // histograms per head
    const Threshold* known;                        // as in launch_select, or nullptr
};

// k - s' and whether anything has to be searched (not all of the candidates are kept, nor none)
__device__ __forceinline__ bool needs_search(int32_t k, int32_t n, int32_t s, uint32_t* m) {
    *m = (uint32_t)(k - s);
    return k > s && *m < (uint32_t)(n - s);
}

// order_key without its top bit
__device__ __forceinline__ uint32_t key31(float x) {
    const int32_t b = __float_as_int(x + 0.0f);                    // -0 -> +0
    return (uint32_t)(b ^ (b >> 31)) & 0x7FFFFFFFu;
}

// Step 1 from scores in memory: workgroup (blockIdx.x, head) counts an equal share of the head.
__global__ __launch_bounds__(kSplitThreads) void split_hist_kernel(SplitArgs a) {
    __shared__ uint32_t hist[kRawHistWords];
    const int head = blockIdx.y, tid = threadIdx.x;
    const int32_t n = a.n, s = a.n_sink < n ? a.n_sink : n;
    uint32_t m;
    if (!needs_search((int32_t)(a.offsets[head + 1] - a.offsets[head]), n, s, &m)) return;
    if (a.known && a.known[head].key31 != kNoThreshold) return;
    const int32_t part = (n + a.hists - 1) / a.hists;
    const int32_t j0 = (int32_t)blockIdx.x * part;
    const int32_t j1 = j0 + part < n ? j0 + part : n;
    const float* sc = a.scores + (size_t)head * n;
    for (int i = tid; i < kRawHistWords; i += kSplitThreads) hist[i] = 0;
    __syncthreads();
    constexpr int kU = 8;
    for (int32_t b = j0; b < j1; b += kU * kSplitThreads) {
        float v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t j = b + u * kSplitThreads + tid;
            v[u] = sc[j < j1 ? j : j1 - 1];        // (not as a branch, or each load is waited for inside it)
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t j = b + u * kSplitThreads + tid;
            // by the key, as the flags of step 2: the two agree whatever the caller's scores are
            if (j >= s && j < j1) raw_hist_count(hist, __uint_as_float(key31(v[u])));
        }
    }
    __syncthreads();
    raw_hist_store<kSplitThreads>(hist, a.ws.hist, a.ws.coarse, head * a.ws.hists + blockIdx.x);
}

// The bin in which the running count from the top of 64*PER counts reaches `want`: called by one
// wave, lane L holds counts 64*PER-1 - (L*PER + i) in c[i].  The lane that finds it writes
// {bin, want left inside it} to LDS.  Returns the sum of all counts.
template <int PER>
__device__ __forceinline__ uint32_t wave_find(const uint32_t (&c)[PER], uint32_t want, uint32_t* out) {
    const int lane = threadIdx.x & 63;
    uint32_t tot = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) tot += c[i];
    uint32_t incl = wave_inclusive(tot);
    uint32_t run = incl - tot;
    if (run < want && want <= incl) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (want <= run + c[i]) { out[0] = (uint32_t)(64 * PER - 1 - (lane * PER + i)); out[1] = want - run; break; }
            run += c[i];
        }
    }
    return (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
}

// KNOWN: a.known is given.
template <bool KNOWN>
__global__ __launch_bounds__(kSplitThreads) void split_flag_kernel(SplitArgs a) {
    __shared__ uint32_t exps[256], fine[64], found[2];
    const int head = blockIdx.x, x0 = blockIdx.y;  // (a head's workgroups, which read the same data, in one L2: launch_gather)
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t n = a.n, s = a.n_sink < n ? a.n_sink : n;
    const int64_t o0 = a.offsets[head], o1 = a.offsets[head + 1];
    const int32_t j0 = (int32_t)x0 * a.part;
    const int32_t j1 = j0 + a.part < n ? j0 + a.part : n;
    float* sc = a.scores + (size_t)head * n;
    // all of the first loads go out together, before anything is decided
    const uint32_t given = KNOWN ? a.known[head].key31 : kNoThreshold;
    uint32_t ce = 0;                               // thread (half, exponent): half of the histograms each
    const uint32_t* co = a.ws.coarse + (size_t)head * a.ws.hists * 256 + (tid & 255);
    if (!KNOWN || given == kNoThreshold) {
        // (sixteen loads at a time, clamped instead of branched around)
        for (int h0 = tid >> 8; h0 < a.hists; h0 += 32) {
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int h = h0 + 2 * u;
                const uint32_t c = co[(h < a.hists ? h : h0) * 256];
                ce += h < a.hists ? c : 0u;
            }
        }
    }
    constexpr int kU = 8;
    float v[kU];
    auto load = [&](int32_t b) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t j = b + u * kSplitThreads + tid;
            v[u] = j < j1 ? sc[j] : 0.f;
        }
    };
    uint32_t m;
    const bool search = needs_search((int32_t)(o1 - o0), n, s, &m);
    const bool write = a.scale_blocks > 0 && a.write_scaled;
    if (!search && !write) return;
    load(j0);
    const HeadScale scale = head_scale(head_partial(a.partial + (size_t)head * kMaxBlocksPerHead, a.scale_blocks), a.scale_blocks, n);
    uint32_t lo = given, hi = given;
    if (KNOWN && search && given != kNoThreshold) {
        if (x0 == 0 && tid == 0) a.ws.range[head] = uint2{lo, hi};
    } else if (search) {
        if (tid < 64) fine[tid] = 0;
        if (tid < 256) exps[tid] = ce;
        __syncthreads();
        if (tid >= 256) atomicAdd(&exps[tid & 255], ce);
        __syncthreads();
        if (tid < 64) {
            const uint32_t c[4] = {exps[255 - 4 * lane], exps[254 - 4 * lane], exps[253 - 4 * lane], exps[252 - 4 * lane]};
            // step 3 takes for granted that the range holds the cut: if counts went missing, everything is in it
            if (wave_find<4>(c, m, found) != (uint32_t)(n - s) && lane == 0) { found[0] = 255u; found[1] = 1u; }
        }
        __syncthreads();
        const uint32_t ex = found[0], want = found[1];
        for (int i = tid; i < a.hists * 16; i += kSplitThreads) {       // a thread per histogram and bin of the exponent
            const uint32_t bin = ex * 16 + (i & 15);
            const uint32_t w = a.ws.hist[((size_t)head * a.ws.hists + (i >> 4)) * kRawHistWords + (bin >> 1)];
            atomicAdd(&fine[i & 15], (bin & 1u) ? w >> 16 : w & 0xFFFFu);
        }
        __syncthreads();
        if (tid < 64) {
            const uint32_t c[1] = {fine[63 - lane]};
            wave_find<1>(c, want, found);
        }
        __syncthreads();
        const uint32_t bin = ex * 16 + (found[0] & 15u);
        lo = key31(scale(__uint_as_float(bin << kRawShift)));
        hi = key31(scale(__uint_as_float((bin << kRawShift) | ((1u << kRawShift) - 1u))));
        if (ex >= 255u) { lo = 0u; hi = 0x7FFFFFFFu; }                      // beyond the finite range: everything
        if (scale.on && scale.zero) lo = hi = key31(scale.uniform);         // all scores are this one
        if (x0 == 0 && tid == 0) a.ws.range[head] = uint2{lo, hi};
    }
    unsigned long long* g = a.ws.gmask + (size_t)head * a.ws.words;
    unsigned long long* e = a.ws.emask + (size_t)head * a.ws.words;
    for (int32_t b = j0; b < j1; b += kU * kSplitThreads) {
        if (b > j0) load(b);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t j = b + u * kSplitThreads + tid;
            const float x = scale(v[u]);
            if (write && j < j1) sc[j] = x;
            if (search) {
                const bool cd = j >= s && j < j1;
                const uint32_t k = key31(x);
                const unsigned long long bg = __ballot(cd && k > hi), be = __ballot(cd && k >= lo && k <= hi);
                const int32_t w0 = j - lane;       // first token of the wave's word
                if (lane == 0 && w0 < j1) { g[w0 >> 6] = bg; e[w0 >> 6] = be; }
            }
        }
    }
}

constexpr int kWideBits = 10, kWideDigits = 1 << kWideBits;   // digits of a list in LDS

struct EmitShared {
    unsigned long long gmask[kSplitMaxWords];      // kept tokens
    unsigned long long emask[kSplitMaxWords];      // candidates in the range, then those equal to the threshold
    union {
        struct {
            uint32_t pairs[2 * kSplitPairs];       // (key - lo, token) of the candidates in the range,
            alignas(16) uint32_t wpos[kSplitMaxWords];     // counts of their digits; later: output position of a word's first kept token
        };
        uint16_t list[kSplitList];                 // or the candidates' tokens, ascending, without bit 16
    };
    alignas(16) uint32_t hist[256];
    uint32_t wave_tot[2][kSplitWaves];
    uint32_t digit, want, count;
    uint32_t low;                                  // place in the list of the first token from 65536 on
};

// exclusive prefix of x over the workgroup's threads; the total goes to *total
__device__ __forceinline__ uint32_t block_exclusive(uint32_t x, uint32_t* wave_tot, uint32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = wave_inclusive(x);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
        const uint32_t t = wave_tot[w];
        before += w < wave ? t : 0u;
        all += t;
    }
    *total = all;
    return before + incl - x;
}

// Counts a digit per lane in hist (LDS); lanes of the same digit as the first one, as equal scores have, in
// one addition.  All 64 lanes must be there.
__device__ __forceinline__ void count_digit(uint32_t* hist, uint32_t digit, bool counts) {
    const unsigned long long all = __ballot(counts);
    if (!all) return;
    const int leader = __ffsll(all) - 1;
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)digit, leader);
    const unsigned long long same = __ballot(counts && digit == first);
    if ((threadIdx.x & 63) == leader) atomicAdd(&hist[first], (uint32_t)__popcll(same));
    else if (counts && digit != first) atomicAdd(&hist[digit], 1u);
}

// One digit of the search for the threshold: hist[0..VALUES-1] counts the digit's values (zeroed
// again), *want becomes the rank inside the chosen value, *count that value's count.  Ends with a barrier.
template <int VALUES = 256>
__device__ __forceinline__ void pick_digit(uint32_t* hist, uint32_t* digit, uint32_t* want, uint32_t* count) {
    constexpr int kPer = VALUES / 64;
    if (threadIdx.x < 64) {                        // lane L looks at values VALUES-1-kPer*L and down
        const int lane = threadIdx.x;
        uint32_t c[kPer], tot = 0;
#pragma unroll
        for (int i = 0; i < kPer; i += 4) {
            uint4& four = reinterpret_cast<uint4*>(hist)[(VALUES - 4 - kPer * lane - i) / 4];
            const uint4 v = four;
            four = uint4{0, 0, 0, 0};
            c[i] = v.w; c[i + 1] = v.z; c[i + 2] = v.y; c[i + 3] = v.x;
            tot += (v.x + v.y) + (v.z + v.w);
        }
        uint32_t incl = wave_inclusive(tot);
        uint32_t run = incl - tot;
        const uint32_t w = *want;
        if (run < w && w <= incl) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                if (w <= run + c[i]) { *digit = VALUES - 1 - kPer * lane - i; *want = w - run; *count = c[i]; break; }
                run += c[i];
            }
        }
    }
    __syncthreads();
}

// ROW_U4 > 0: the workgroup also copies its share's rows of K and V (gather step of Algorithm 1);
// share <= kSplitShare then.  KNOWN: budgets and thresholds come from the budget allocation, on the device: a workgroup's share is
// the head's rows by the workgroups, listed kSplitShare at a time where it copies them.
template <int ROW_U4, bool KNOWN>
__global__ __launch_bounds__(kSplitThreads) void split_emit_kernel(SplitArgs a, int32_t* __restrict__ indices, int share,
                                                                   GatherArgs ga, int heads_x) {
    __shared__ EmitShared sm;
    __shared__ int32_t stage[ROW_U4 ? kSplitShare : 1];
    const int head = heads_x ? blockIdx.x : blockIdx.y, x0 = heads_x ? blockIdx.y : blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t n = a.n, s = a.n_sink < n ? a.n_sink : n;
    const int64_t o0 = a.offsets[head], o1 = a.offsets[head + 1];
    // all of the first loads go out together, before anything is decided
    const int words = (n + 63) >> 6;
    const int w0 = tid * kSplitWordsPerThread;
    unsigned long long g[kSplitWordsPerThread], e[kSplitWordsPerThread];
    {
        const unsigned long long* gp = a.ws.gmask + (size_t)head * a.ws.words;
        const unsigned long long* ep = a.ws.emask + (size_t)head * a.ws.words;
#pragma unroll
        for (int i = 0; i < kSplitWordsPerThread; ++i) {
            g[i] = w0 + i < words ? gp[w0 + i] : 0ull;
            e[i] = w0 + i < words ? ep[w0 + i] : 0ull;
        }
    }
    const uint2 range = a.ws.range[head];
    const int scale_blocks = a.write_scaled ? 0 : a.scale_blocks;
    const HeadScale scale = head_scale(head_partial(a.partial + (size_t)head * kMaxBlocksPerHead, scale_blocks), scale_blocks, n);
    const float* sc = a.scores + (size_t)head * n;
    const int32_t k = (int32_t)(o1 - o0);
    const int shares = (int)(heads_x ? gridDim.y : gridDim.x);
    if (KNOWN) share = (k + shares - 1) / shares;
    const int32_t begin = (int32_t)x0 * share;
    const int32_t end = begin + share < k ? begin + share : k;     // output rows begin .. end-1 are this workgroup's
    uint32_t m;
    const bool search = needs_search(k, n, s, &m);
    if (begin >= end) return;
    int32_t* out = indices + o0;
    // rows r0 .. r1-1 are being listed: all of them, or as many as the stage takes
    constexpr bool kPieces = KNOWN && ROW_U4 > 0;
    int32_t r0 = begin, r1 = kPieces && end - begin > kSplitShare ? begin + kSplitShare : end;
    auto put = [&](int32_t p, int32_t j) {                         // row p of the head is token j
        if (ROW_U4) stage[p - r0] = j; else out[p] = j;
    };
    auto next = [&]() {
        if (!kPieces) return false;
        r0 = r1;
        r1 = end - r0 > kSplitShare ? r0 + kSplitShare : end;
        if (r0 < end) __syncthreads();                             // the stage has been read
        return r0 < end;
    };
    auto gather = [&]() {
        if constexpr (ROW_U4 > 0) {
            __syncthreads();
            for (int32_t p = r0 + tid; p < r1; p += kSplitThreads) out[p] = stage[p - r0];
            constexpr int kRows = kSplitThreads / ROW_U4, kFlight = 8;     // rows per instruction, and in flight per thread
            const int c = tid % ROW_U4, rsub = tid / ROW_U4;
            const int32_t count = r1 - r0;
#pragma unroll 1
            for (int which = 0; which < 2; ++which) {
                const u32x4* src = (which ? ga.V : ga.K) + (size_t)head * n * ROW_U4 + c;
                u32x4* dst = (which ? ga.V_out : ga.K_out) + (size_t)(o0 + r0) * ROW_U4 + c;
#pragma unroll 1
                for (int32_t p0 = 0; p0 < count; p0 += kRows * kFlight) {
                    u32x4 v[kFlight];
#pragma unroll
                    for (int it = 0; it < kFlight; ++it) {
                        const int32_t p = p0 + it * kRows + rsub;
                        const uint32_t j = (uint32_t)stage[p < count ? p : count - 1];
                        // every place holds a token by construction; never read outside the cache whatever the scores were
                        v[it] = __builtin_nontemporal_load(src + (size_t)(j < (uint32_t)n ? j : 0u) * ROW_U4);
                    }
#pragma unroll
                    for (int it = 0; it < kFlight; ++it) {
                        const int32_t p = p0 + it * kRows + rsub;
                        if (p < count) __builtin_nontemporal_store(v[it], dst + (size_t)p * ROW_U4);
                    }
                }
            }
        }
    };
    if (!search) {                                                 // tokens 0 .. k-1: sinks only, or everything
        do {
            for (int32_t j = r0 + tid; j < r1; j += kSplitThreads) put(j, j);
            gather();
        } while (next());
        return;
    }
    // ---- the bitmaps -------------------------------------------------------------------------------
    uint32_t ng = 0, ne = 0, total_g, total_e;
#pragma unroll
    for (int i = 0; i < kSplitWordsPerThread; ++i) {
        ng += (uint32_t)__popcll(g[i]);
        ne += (uint32_t)__popcll(e[i]);
        sm.gmask[w0 + i] = g[i];
        sm.emask[w0 + i] = e[i];
    }
    for (int i = tid; i < 256; i += kSplitThreads) sm.hist[i] = 0;
    for (int i = tid; i < kWideDigits; i += kSplitThreads) sm.wpos[i] = 0;
    uint32_t slot;
    {   // both sums behind one barrier
        const uint32_t ig = wave_inclusive(ng), ie = wave_inclusive(ne);
        if (lane == 63) { sm.wave_tot[0][wave] = ig; sm.wave_tot[1][wave] = ie; }
        __syncthreads();
        uint32_t before = 0;
        total_g = total_e = 0;
#pragma unroll
        for (int w = 0; w < kSplitWaves; ++w) {
            before += w < wave ? sm.wave_tot[1][w] : 0u;
            total_g += sm.wave_tot[0][w];
            total_e += sm.wave_tot[1][w];
        }
        slot = before + ie - ne;
    }
    uint32_t need = m - total_g;                                   // how many of the range are kept (>= 1)
    // ---- the threshold among the keys in the range ---------------------------------------------------
    const uint32_t width = range.y - range.x;
    int rem = width ? 32 - __clz((int)width) : 0;                  // bits of key - lo not yet decided
    if (need < total_e && rem > 0) {
        uint32_t fixed = 0;
        if (tid == 0) sm.want = need;
        if (total_e > (uint32_t)kSplitList) {
            // digit by digit from memory until the rest fits the list, then one pass that keeps what is above and leaves
            // the rest flagged (8 heads of 131072 equal scores, a tenth kept, curdkv_select: 450 -> 210 us)
            // f(word, token is in the range, its key - lo), a wave per word, kU words' scores and flags in flight
            auto for_each_in_range = [&](auto f) {
                constexpr int kU = 32;
                const uint32_t* half = reinterpret_cast<const uint32_t*>(sm.emask) + (lane >> 5);
                for (int wb = wave * kU; wb < words; wb += kSplitWaves * kU) {
                    float x[kU];
                    uint32_t mine[kU];
#pragma unroll
                    for (int u = 0; u < kU; ++u) {
                        const int32_t j = (wb + u) * 64 + lane;
                        x[u] = sc[j < n ? j : n - 1];
                        mine[u] = half[2 * (wb + u)];              // (zero beyond the head)
                    }
#pragma unroll
                    for (int u = 0; u < kU; ++u) f(wb + u, ((mine[u] >> (lane & 31)) & 1u) != 0, key31(scale(x[u])) - range.x);
                }
            };
            __syncthreads();
            while (rem > 0 && total_e > (uint32_t)kSplitList) {
                const int w = rem < 8 ? rem : 8, shift = rem - w;
                for_each_in_range([&](int, bool mine, uint32_t key) {
                    count_digit(sm.hist, (key >> shift) & ((1u << w) - 1u), mine && (key >> rem) == fixed);
                });
                __syncthreads();
                pick_digit(sm.hist, &sm.digit, &sm.want, &sm.count);
                fixed = (fixed << w) | sm.digit;
                total_e = sm.count;
                rem = shift;
            }
            for_each_in_range([&](int w1, bool mine, uint32_t key) {
                const unsigned long long above = __ballot(mine && (key >> rem) > fixed), rest = __ballot(mine && (key >> rem) == fixed);
                if (lane == 0) { atomicOr(&sm.gmask[w1], above); sm.emask[w1] = rest; }
            });
            __syncthreads();
            ne = 0;
#pragma unroll
            for (int i = 0; i < kSplitWordsPerThread; ++i) {
                e[i] = sm.emask[w0 + i];
                ne += (uint32_t)__popcll(e[i]);
            }
            slot = block_exclusive(ne, sm.wave_tot[1], &total_e);
        }
        if (rem > 0 && total_e <= (uint32_t)kSplitPairs) {         // tokens first, then all their keys at once
#pragma unroll
            for (int i = 0; i < kSplitWordsPerThread; ++i)
                for (unsigned long long x = e[i]; x; x &= x - 1) sm.pairs[2 * slot++ + 1] = (uint32_t)((w0 + i) * 64 + __ffsll(x) - 1);
            __syncthreads();
            for (uint32_t i = tid; i < total_e; i += kSplitThreads) sm.pairs[2 * i] = key31(scale(sc[sm.pairs[2 * i + 1]])) - range.x;
            __syncthreads();
            while (rem > 0) {                                      // ten bits at a time: two digits of a range of a sixteenth of a binade
                const int w = rem < kWideBits ? rem : kWideBits, shift = rem - w;
                for (uint32_t i = tid; i < total_e; i += kSplitThreads) {
                    const uint32_t key = sm.pairs[2 * i];
                    if ((key >> rem) == fixed) atomicAdd(&sm.wpos[(key >> shift) & ((1u << w) - 1u)], 1u);
                }
                __syncthreads();
                pick_digit<kWideDigits>(sm.wpos, &sm.digit, &sm.want, &sm.count);
                fixed = (fixed << w) | sm.digit;
                rem = shift;
            }
            // the list's members above the threshold join the kept ones, those equal to it stay flagged
            for (uint32_t i = tid; i < total_e; i += kSplitThreads) {
                const uint32_t key = sm.pairs[2 * i], j = sm.pairs[2 * i + 1];
                if (key > fixed) atomicOr(&sm.gmask[j >> 6], 1ull << (j & 63u));
                if (key != fixed) atomicAnd(&sm.emask[j >> 6], ~(1ull << (j & 63u)));
            }
            __syncthreads();
        } else if (rem > 0) {                                      // tokens in LDS, keys in registers
            if (w0 == 65536 / 64) sm.low = slot;
#pragma unroll
            for (int i = 0; i < kSplitWordsPerThread; ++i)
                for (unsigned long long x = e[i]; x; x &= x - 1) sm.list[slot++] = (uint16_t)((w0 + i) * 64 + __ffsll(x) - 1);
            __syncthreads();
            const uint32_t low = sm.low;
            auto token = [&](uint32_t p) { return (uint32_t)sm.list[p] | (p >= low ? 65536u : 0u); };
            constexpr int kGroup = 8;                              // keys of a thread fetched together
            uint32_t key[kSplitList / kSplitThreads];
#pragma unroll
            for (int u0 = 0; u0 < kSplitList / kSplitThreads; u0 += kGroup) {
                if ((uint32_t)(u0 * kSplitThreads) < total_e) {
                    float x[kGroup];
#pragma unroll
                    for (int u = 0; u < kGroup; ++u) {
                        const uint32_t p = (uint32_t)((u0 + u) * kSplitThreads + tid);
                        x[u] = sc[token(p < total_e ? p : total_e - 1)];
                    }
#pragma unroll
                    for (int u = 0; u < kGroup; ++u) {
                        const uint32_t p = (uint32_t)((u0 + u) * kSplitThreads + tid);
                        key[u0 + u] = p < total_e ? key31(scale(x[u])) - range.x : 0xFFFFFFFFu;   // (nobody's digits)
                    }
                }
            }
            // f(number in the list, key - lo)
            auto for_each_listed = [&](auto f) {
#pragma unroll
                for (int u = 0; u < kSplitList / kSplitThreads; ++u) {
                    int count = __builtin_amdgcn_readfirstlane((int)total_e);
                    asm volatile("" : "+s"(count));                // or 32 comparisons are kept in scalar registers from the start
                    if (u * kSplitThreads < count) f((uint32_t)(u * kSplitThreads + tid), key[u]);
                }
            };
            while (rem > 0) {
                const int w = rem < 8 ? rem : 8, shift = rem - w;
                for_each_listed([&](uint32_t, uint32_t k1) { count_digit(sm.hist, (k1 >> shift) & ((1u << w) - 1u), (k1 >> rem) == fixed); });
                __syncthreads();
                pick_digit(sm.hist, &sm.digit, &sm.want, &sm.count);
                fixed = (fixed << w) | sm.digit;
                rem = shift;
            }
            for_each_listed([&](uint32_t p, uint32_t k1) {
                if (p < total_e && k1 != fixed) {
                    const uint32_t j = token(p);
                    if (k1 > fixed) atomicOr(&sm.gmask[j >> 6], 1ull << (j & 63u));
                    atomicAnd(&sm.emask[j >> 6], ~(1ull << (j & 63u)));
                }
            });
            __syncthreads();
        }
        need = sm.want;                                            // keys equal to the threshold still to be kept
#pragma unroll
        for (int i = 0; i < kSplitWordsPerThread; ++i) { g[i] = sm.gmask[w0 + i]; e[i] = sm.emask[w0 + i]; }
    }
    // ---- the first `need` flagged tokens join the kept ones; output positions -------------------------
    ne = 0;
#pragma unroll
    for (int i = 0; i < kSplitWordsPerThread; ++i) ne += (uint32_t)__popcll(e[i]);
    __syncthreads();                                               // the totals have been read by everyone
    uint32_t eq_before = block_exclusive(ne, sm.wave_tot[0], &total_e), nk = 0;
#pragma unroll
    for (int i = 0; i < kSplitWordsPerThread; ++i) {
        const uint32_t c = (uint32_t)__popcll(e[i]);
        unsigned long long keep = e[i];
        if (eq_before >= need) keep = 0ull;                        // quota already used up
        else if (eq_before + c > need)                             // the word where it runs out
            for (uint32_t drop = eq_before + c - need; drop; --drop) keep &= ~(1ull << (63 - __clzll((long long)keep)));
        eq_before += c;
        g[i] |= keep;
        nk += (uint32_t)__popcll(g[i]);
    }
    uint32_t pos = (uint32_t)s + block_exclusive(nk, sm.wave_tot[1], &total_g);
#pragma unroll
    for (int i = 0; i < kSplitWordsPerThread; ++i) {
        sm.gmask[w0 + i] = g[i];
        sm.wpos[w0 + i] = pos;
        pos += (uint32_t)__popcll(g[i]);
    }
    __syncthreads();
    // ---- this workgroup's share ----------------------------------------------------------------------------
    do {
    for (int32_t j = r0 + tid; j < r1 && j < s; j += kSplitThreads) put(j, j);
    // only the words that hold rows r0 .. r1-1: positions ascend, so a search finds the first one, and the pass ends behind the last.  (All
    // words, digits of 8 bits, a barrier per sum and 8 of a histogram's counts in flight in split_flag_kernel: one call for 8 heads of 131072 tokens
    // 119.2 us, so 116.4, 1 head 36.2 and 34.4, 8 of 60000 66.8 and 64.7; curdkv_select of 8 of 131072 21.0 and 20.0.)
    int lo = 0;
    for (int step = kSplitMaxWords / 2; step > 0; step >>= 1)
        if (lo + step < words && (int32_t)sm.wpos[lo + step] <= r0) lo += step;
    for (int q = lo * 4 + tid; q < words * 4; q += kSplitThreads) {        // a thread per quarter word (16 tokens)
        if ((int32_t)sm.wpos[q >> 2] >= r1) break;
        const int w = q >> 2, part = q & 3;
        const unsigned long long word = sm.gmask[w];
        uint32_t mm = (uint32_t)(word >> (16 * part)) & 0xFFFFu;
        int32_t p = (int32_t)sm.wpos[w] + (int32_t)__popcll(word & ((1ull << (16 * part)) - 1ull));
        if (p >= r1 || p + 16 <= r0) continue;
        while (mm) {
            const int bit = __ffs(mm) - 1;
            mm &= mm - 1;
            if (p >= r0 && p < r1) put(p, w * 64 + 16 * part + bit);
            ++p;
        }
    }
    gather();
    } while (next());
}

// Which heads take this route, where select_gather_kernel does not.  One call, this against one workgroup per head (us): 1 head of 32768
// tokens 31 against 33, 8 heads 47 against 50, 32 heads 133 against 137; 8 heads of 16384 33.8 against 32, 64 heads
// of 32768 247 against 246: hence 24576 and 32 heads.  Longer heads would otherwise be streamed twice by one
// workgroup (8 heads of 131072 tokens: 188 -> 136, 1 head 157 -> 54, 64 heads 933 -> 902, 256 heads no
// difference).  The separate selection needs a launch more (32 heads of 32768: 147 against 137 for the three
// calls), so it stays with one workgroup as long as its registers hold the head.
bool split_wanted(const curdkv_ctx* ctx) { return ctx->cfg.max_tokens > kSplitMinTokens && ctx->heads <= kSplitMaxHeads; }

bool split_applicable(const curdkv_ctx* ctx, int64_t n, bool one_call) {
    if (!ctx->d_split_ws || n > kSplitMaxTokens) return false;
    return n > (one_call && ctx->heads <= 32 ? kSplitMinTokens : kSplitMinTokensElse);
}

// One or two long heads are better scored by more workgroups each than there are histograms, which are then made from
// memory, a launch more.  One call, us, at most 64 workgroups a head that count and as many as there are units: 1 head of 131072
// tokens 50.6 and 36.8; 2 heads of 32768 26.9 and 27.6, of 65536 37.7 and 36.9, of 131072 59.8 and 53.3; 3 heads
// put 192 workgroups on the chip as it is.
bool split_counts_in_scan(const curdkv_ctx* ctx, int64_t n) { return ctx->heads > 2 || n <= (int64_t)ctx->heads * kSplitMinTokens; }

uint32_t* split_hist(const curdkv_ctx* ctx) { return carve(ctx).hist; }
uint32_t* split_coarse(const curdkv_ctx* ctx) { return carve(ctx).coarse; }

// One-call path: whether step 3 should gather as well.  It saves a launch and the indices' trip
// through memory; the stand-alone gather kernel's many small workgroups move long lists faster.
static bool emit_gathers(const curdkv_ctx* ctx, int64_t total) { return total <= (int64_t)ctx->num_cu * 1024; }

hipError_t launch_split_select(const curdkv_ctx* ctx, float* scores, int64_t n, int32_t n_sink,
                               const int64_t* d_offsets, int64_t max_budget, int64_t total, int32_t* indices, hipStream_t stream,
                               int scale_blocks, bool write_scaled, const void* known_thresholds, SelectGather* gather, int hists) {
    SplitArgs a{carve(ctx), scores, (int32_t)n, n_sink, d_offsets, ctx->d_partial, scale_blocks, write_scaled ? 1 : 0, 0, hists,
                static_cast<const Threshold*>(known_thresholds)};
    if (hists == 0) {
        int64_t h = ((int64_t)ctx->num_cu * 2 + ctx->heads - 1) / ctx->heads;
        const int64_t least = (n + 8191) / 8192;
        if (h < least) h = least;
        a.hists = (int)(h < a.ws.hists ? h : a.ws.hists);
        split_hist_kernel<<<dim3((unsigned)a.hists, (unsigned)ctx->heads), kSplitThreads, 0, stream>>>(a);
    }
    int64_t parts = ((int64_t)ctx->num_cu * 2 + ctx->heads - 1) / ctx->heads;
    int64_t part = (n + parts - 1) / parts;
    if (part > 16384) part = 16384;
    a.part = (int)((part + kSplitThreads - 1) / kSplitThreads * kSplitThreads);
    const dim3 parts_grid((unsigned)ctx->heads, (unsigned)((n + a.part - 1) / a.part));
    if (a.known) split_flag_kernel<true><<<parts_grid, kSplitThreads, 0, stream>>>(a);
    else split_flag_kernel<false><<<parts_grid, kSplitThreads, 0, stream>>>(a);
    const bool with_gather = gather && gather->total > 0 && emit_gathers(ctx, gather->total);
    // shares such that there are about two workgroups per compute unit, or one for lists alone: each resolves the
    // threshold of its head again, which two of a unit do no sooner than one after the other.  With 4096 rows each whatever their number,
    // curdkv_select of 100 heads of 41943 tokens, 70 % kept, 42.3 us, so 36.4; of 64 heads of 65536 normal rows, 30 %, 47.8 and 42.3.
    int64_t share;
    if (with_gather) {
        share = (gather->total + ctx->num_cu * 2 - 1) / (ctx->num_cu * 2);
        share = share < 64 ? 64 : share > kSplitShare ? kSplitShare : (share + 31) / 32 * 32;
    } else {
        const int64_t places = ctx->num_cu / ctx->heads > 1 ? ctx->num_cu / ctx->heads : 1;
        share = (max_budget + places - 1) / places;
        if (share < 4096) share = 4096;
    }
    int64_t shares = (max_budget + share - 1) / share;
    if (max_budget < 0) {                          // every workgroup takes an equal share of its head's rows
        shares = (ctx->num_cu * (with_gather ? 2 : 1) + ctx->heads - 1) / ctx->heads;
        share = 0;
    }
    // As in launch_gather (select_kernels.hip).  Lists alone: where heads of one XCD have the large budgets, half kept, one head of 8 with all rows, us, shares and heads along x, 32 heads
    // of 109334 tokens 28.2 and 36.5, 128 of 65536 48.0 and 56.9, 16 of 131072 21.4 and 25.0; equal budgets, over 36 sizes, heads along x 5 % ahead.
    const bool heads_x = even_budgets(ctx, max_budget, total);
    const unsigned each = (unsigned)(shares > 0 ? shares : 1);
    const dim3 grid = heads_x ? dim3((unsigned)ctx->heads, each) : dim3(each, (unsigned)ctx->heads);
    GatherArgs ga{};
    if (with_gather) {
        ga = GatherArgs{(const u32x4*)gather->K, (const u32x4*)gather->V, (u32x4*)gather->K_out, (u32x4*)gather->V_out};
        gather->done = true;
    }
    auto emit = [&](auto known) {
        constexpr bool KNOWN = decltype(known)::value;
        if (!with_gather) split_emit_kernel<0, KNOWN><<<grid, kSplitThreads, 0, stream>>>(a, indices, (int)share, ga, heads_x ? 1 : 0);
        else if (ctx->cfg.dtype == CURDKV_DTYPE_BF16) split_emit_kernel<16, KNOWN><<<grid, kSplitThreads, 0, stream>>>(a, indices, (int)share, ga, heads_x ? 1 : 0);
        else split_emit_kernel<32, KNOWN><<<grid, kSplitThreads, 0, stream>>>(a, indices, (int)share, ga, heads_x ? 1 : 0);
    };
    if (max_budget < 0) emit(std::true_type{});
    else emit(std::false_type{});
    return hipGetLastError();
}

}  // namespace curdkv
