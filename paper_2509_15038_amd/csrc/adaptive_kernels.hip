// AdaCurDKV head-wise budgets (Section 3.2, "Adaptive budget allocation"), for
// gfx950: a layer keeps H*k tokens in all, the top normalised scores across its
// heads, except that every head is guaranteed its own best floor(alpha*k) tokens
// (sinks first).  Only the per-head COUNTS are needed here; feeding them to the
// per-head selection then yields the layer-wide set.
//
// With c_h(t) = number of non-sink tokens of head h that rank above a threshold
// t (ties in (head, token) order), head h keeps max(g, c_h(t)) non-sink tokens,
// g being the guaranteed number, and the threshold is where
//     sum_h max(0, c_h(t) - g) = R,      R = H*(k - s') - H*g.
// The counting functions c_h come from per-head histograms of the order-
// preserving keys over the 4096 bins of the selection (bin12, select_device.h):
//   * the histograms, and their sums per exponent, are made by the fused kernel while it has a
//     head's keys in registers, or by ada_hist_kernel from scores in memory, several workgroups per
//     (layer, head) where heads are few, each a histogram of its part;
//   * ada_cut_kernel, a workgroup per head and part: every workgroup finds the bin in which the sum above reaches R (the same
//     small computation in each of them: first over the layer's sums per exponent, then over the 32 bins of one exponent),
//     and copies its own part's keys inside that bin (a fraction of a percent of the head) to the workspace;
//   * ada_allot_kernel, one workgroup per layer, resolves the remaining key bits on those few keys in LDS, allots keys equal to the
//     threshold head by head, and writes the budgets, their prefix sums and the gather's block table
//     for the layer (every layer keeps H*k rows, so a layer's first row is known).
// Bins too full for the lists (a layer of equal scores, say) and scores of 2 and above
// make the layer's workgroup refine the threshold by reading the layer's scores
// itself, a few bits per pass: slow, and exact all the same.
// No token order is needed anywhere.
//
// What bounds these kernels is latency: loads, barriers and LDS round trips in a chain.  Two launches instead of one whose last workgroup
// of a layer went on: a device-scope fence, which such a hand-over needs, is a cache-wide operation here (eight L2s) and dearer
// than the boundary between two kernels.  With all H histograms of 4096 bins scanned by every workgroup and that hand-over, 8 heads of
// 1024 tokens took 19.6 us, 256 of 32768 29.2; the two kernels take 4.8 + 5.3 and 12.4 + 7.0.  Histograms in parts (8 heads of
// 131072 tokens): 19.4 -> 5.7 us, normalisation (5.1) included.

#include <mutex>

#include "select_device.h"

namespace curdkv {

constexpr int kAdaThreads = 1024;
constexpr int kAdaWaves = kAdaThreads / 64;
constexpr int kAdaU = 8;                          // scores per thread in flight
constexpr int kAdaOwn = 32;                       // cut kernel: scores per thread loaded up front, at most
// In-bin keys a head hands to its layer's workgroup; with more in one head the layer's scores are read again (curdkv_adaptive_budgets, 8 heads of 131072
// tokens 22.7 us with 2040 keys, 704 with 2049).
constexpr int kAdaSeg = 2048;
constexpr int kAdaList = 4096;                    // (key, head) pairs that workgroup resolves in LDS
constexpr int kAdaDigWords = 8192;                // its per-head digit histograms: H << bits words
constexpr int kAdaMaxHeads = 1024;                // kv_heads these kernels are laid out for
constexpr int kAdaSlots = 256;                    // histograms in all, or one per head where there are more
constexpr int kAdaMaxParts = 32;                  // histograms per head
constexpr int kAdaPartTokens = 4096;              // a part is no shorter
constexpr int kExps = kBins12 / 32;               // sums per exponent: 32 bins each

struct AdaWorkspace {                             // device pointers into one allocation
    uint32_t* hist;                               // [heads][parts][4096] bin12 histograms of the candidates
    uint32_t* coarse;                             // [heads][parts][128] their sums per exponent
    uint32_t* seg;                                // [heads][kAdaSeg] keys (31 bits) inside the layer's cut bin
    uint32_t* above;                              // [heads] candidates in bins above the cut bin
    uint32_t* inbin;                              // [heads] candidates inside it
    Threshold* known;                             // [heads] what the selection may take over: the layer's threshold
    AdaLayerState* layer;                         // [layers]
};

// Parts a head is counted in: one per compute unit at most, where heads are fewer than those.
static int parts_for(int heads, int64_t n) {
    int64_t parts = kAdaSlots / heads;
    if (parts > (n + kAdaPartTokens - 1) / kAdaPartTokens) parts = (n + kAdaPartTokens - 1) / kAdaPartTokens;
    return (int)(parts < 1 ? 1 : parts < kAdaMaxParts ? parts : kAdaMaxParts);
}
static size_t slots_for(const curdkv_ctx* ctx) { return (size_t)ctx->heads * parts_for(ctx->heads, ctx->cfg.max_tokens); }

static constexpr size_t workspace_bytes_for(size_t slots, size_t heads, size_t layers) {
    return slots * (size_t)(kBins12 + kExps) * 4 + heads * (size_t)kAdaSeg * 4 + heads * 16 + layers * sizeof(AdaLayerState);
}

static AdaWorkspace carve(void* base, const curdkv_ctx* ctx) {
    const size_t heads = (size_t)ctx->heads, slots = slots_for(ctx);
    AdaWorkspace w;
    w.hist = reinterpret_cast<uint32_t*>(base);
    w.coarse = w.hist + slots * kBins12;
    w.seg = w.coarse + slots * kExps;
    w.above = w.seg + heads * kAdaSeg;
    w.inbin = w.above + heads;
    w.known = reinterpret_cast<Threshold*>(w.inbin + heads);
    w.layer = reinterpret_cast<AdaLayerState*>(w.known + heads);
    return w;
}

// Histogram of a part of a head's candidate keys (tokens sp and up) over the selection's 4096 bins: workgroup head*parts + part.
// scale_blocks > 0: `scores` holds un-normalised products, which are normalised on the way.
__global__ __launch_bounds__(kAdaThreads) void ada_hist_kernel(float* __restrict__ scores, int64_t n, int32_t sp, int parts, int64_t part,
                                                               uint32_t* __restrict__ ws_hist, uint32_t* __restrict__ ws_coarse,
                                                               const float* __restrict__ partial, int scale_blocks) {
    __shared__ __align__(16) uint32_t hist[kBins12];
    const int slot = blockIdx.x, head = slot / parts;
    const int tid = threadIdx.x;
    const int64_t j_begin = (int64_t)(slot - head * parts) * part;
    const int64_t j_end = j_begin + part < n ? j_begin + part : n;
    float* sc = scores + (size_t)head * n;
    float cur[kAdaU], nxt[kAdaU];
    auto load = [&](float (&v)[kAdaU], int64_t j0) {
#pragma unroll
        for (int u = 0; u < kAdaU; ++u) {
            const int64_t j = j0 + (int64_t)u * kAdaThreads;
            v[u] = j < j_end ? sc[j] : 0.f;
        }
    };
    load(cur, j_begin + tid);
    const HeadScale scale = head_scale(head_partial(partial + (size_t)head * kMaxBlocksPerHead, scale_blocks), scale_blocks, n);
    for (int i = tid; i < kBins12; i += kAdaThreads) hist[i] = 0;
    __syncthreads();
    for (int64_t j0 = j_begin + tid; j0 < j_end; j0 += (int64_t)kAdaU * kAdaThreads) {
        const int64_t jn = j0 + (int64_t)kAdaU * kAdaThreads;
        if (jn < j_end) load(nxt, jn);
#pragma unroll
        for (int u = 0; u < kAdaU; ++u) {
            const int64_t j = j0 + (int64_t)u * kAdaThreads;
            if (j < j_end) {
                const float v = scale(cur[u]);
                if (scale.on) sc[j] = v;
                if (j >= sp) atomicAdd(&hist[bin12(order_key(v))], 1u);
            }
        }
#pragma unroll
        for (int u = 0; u < kAdaU; ++u) cur[u] = nxt[u];
    }
    __syncthreads();
    hist12_store<kAdaThreads>(hist, ws_hist + (size_t)slot * kBins12, ws_coarse + (size_t)slot * kExps);
}

constexpr int kAdaHeadsAtOnce = kAdaThreads / kExps;             // 8: a thread per head and exponent

// KPT: scores per thread loaded up front.
template <int KPT>
__global__ __launch_bounds__(kAdaThreads) void ada_cut_kernel(AdaWorkspace ws, const float* __restrict__ scores, int64_t n, int H,
                                                              int32_t sp, int32_t g, long long R, int parts, int64_t part) {
    __shared__ uint32_t cum[kAdaHeadsAtOnce][kExps];             // keys of a head in exponents from the top to the i-th
    __shared__ uint32_t fine[kAdaHeadsAtOnce][32];               // the same over the bins of one exponent
    __shared__ uint32_t wave_tot[kAdaWaves], own[33], first[2], count;
    const int head = blockIdx.x / parts, q = blockIdx.x - head * parts;
    const int layer = head / H, my = head - layer * H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t j_begin = (int64_t)q * part;
    const int64_t j_end = j_begin + part < n ? j_begin + part : n;
    const uint32_t len = j_begin < j_end ? (uint32_t)(j_end - j_begin) : 0u;
    const float* sc = scores + (size_t)head * n + j_begin;

    // the sums per exponent are wanted first, then this part's own scores, which arrive while those are being worked on
    auto load_counts = [&](int h0) -> uint32_t {
        const int h = h0 + (tid >> 7);
        if (h >= H) return 0u;
        const uint32_t* c = ws.coarse + (size_t)(layer * H + h) * parts * kExps + (kExps - 1 - (tid & 127));
        uint32_t sum = 0;
#pragma unroll 8
        for (int p = 0; p < parts; ++p) sum += c[p * kExps];
        return sum;
    };
    auto accumulate = [&](uint32_t sum) {                        // fills cum
        uint32_t incl = wave_inclusive(sum);
        if (lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        if (wave & 1) incl += wave_tot[wave - 1];                // (two waves a head)
        cum[tid >> 7][tid & 127] = incl;
        __syncthreads();
    };
    const uint32_t counts = load_counts(0);
    if (len == 0) return;                          // (no part is empty by the launcher's rule)
    float v[KPT];
#pragma unroll
    for (int u = 0; u < KPT; ++u) {                // (not as a branch, or each load is waited for inside it)
        const uint32_t o = (uint32_t)(u * kAdaThreads + tid);
        v[u] = sc[o < len ? o : len - 1];
    }
    // ---- the exponent in which sum_h max(0, c_h - g) reaches R ------------------------------------
    unsigned long long E = 0;
    for (int h0 = 0; h0 < H; h0 += kAdaHeadsAtOnce) {
        accumulate(h0 == 0 ? counts : load_counts(h0));
        if (tid < kExps) {
            const int m = H - h0 < kAdaHeadsAtOnce ? H - h0 : kAdaHeadsAtOnce;
            for (int j = 0; j < m; ++j) {
                const uint32_t c = cum[j][tid];
                if (c > (uint32_t)g) E += c - (uint32_t)g;
            }
        }
    }
    if (wave < 2) {
        const unsigned long long m = __ballot(E >= (unsigned long long)R);
        if (lane == 0) first[wave] = m ? (uint32_t)(wave * 64 + __ffsll(m) - 1) : (uint32_t)(kExps - 1);
    }
    __syncthreads();
    // (the lowest bin always reaches R for histograms of n - sp candidates per head; the bounds
    // keep everything below in range whatever the workspace held)
    const int pos = (int)(first[0] < first[1] ? first[0] : first[1]);
    // ---- the bin of that exponent --------------------------------------------------------------------
    E = 0;
    for (int h0 = 0; h0 < H; h0 += kAdaHeadsAtOnce) {
        if (H > kAdaHeadsAtOnce) accumulate(load_counts(h0));
        const int j = (tid >> 5) & 7, i = tid & 31, slice = tid >> 8, h = h0 + j;      // four slices of the parts
        uint32_t f = 0;
        if (h < H) {
            const uint32_t* c = ws.hist + (size_t)(layer * H + h) * parts * kBins12 + ((kExps - 1 - pos) * 32 + 31 - i);
#pragma unroll 8
            for (int p = slice; p < parts; p += 4) f += c[(size_t)p * kBins12];
        }
        if (slice == 0) fine[j][i] = f;
        if (parts > 1) {
            __syncthreads();
            if (slice > 0 && f) atomicAdd(&fine[j][i], f);
            __syncthreads();
        }
        if (slice == 0) {
            uint32_t incl = wave_inclusive(fine[j][i]);
            const uint32_t low = (uint32_t)__builtin_amdgcn_readlane((int)incl, 31);
            incl -= lane >= 32 ? low : 0u;
            const uint32_t before = pos > 0 ? cum[j][pos - 1] : 0u;
            fine[j][i] = before + incl;
            if (h == my) {
                own[i + 1] = before + incl;
                if (i == 0) own[0] = before;
            }
        }
        __syncthreads();
        if (tid < 32) {
            const int m = H - h0 < kAdaHeadsAtOnce ? H - h0 : kAdaHeadsAtOnce;
            for (int jj = 0; jj < m; ++jj) {
                const uint32_t c = fine[jj][tid];
                if (c > (uint32_t)g) E += c - (uint32_t)g;
            }
        }
    }
    if (wave == 0) {
        const unsigned long long m = __ballot(lane < 32 && E >= (unsigned long long)R);
        if (lane == 0) first[0] = m ? (uint32_t)(__ffsll(m) - 1) : 31u;
    }
    __syncthreads();
    const int i0 = (int)first[0];
    const uint32_t bstar = (uint32_t)((kExps - 1 - pos) * 32 + 31 - i0);
    const uint32_t above_my = own[i0], inbin_my = own[i0 + 1] - own[i0];
    if (tid == 0 && q == 0) {
        ws.above[head] = above_my;
        ws.inbin[head] = inbin_my;
        if (my == 0) ws.layer[layer].bin = bstar;
    }
    // ---- hand this part's keys inside the bin to the layer ----------------------------------------
    if (bstar >= (uint32_t)(kBins12 - 1) || inbin_my > (uint32_t)kAdaSeg) return;
    if (wave == 0) {                               // behind those of the parts before
        uint32_t before = lane < q ? ws.hist[((size_t)head * parts + lane) * kBins12 + bstar] : 0u;
        before = wave_inclusive(before);
        if (lane == 63) count = before;
    }
    __syncthreads();
    uint32_t* seg = ws.seg + (size_t)head * kAdaSeg;
    auto hand_in = [&](float x, bool cand) {
        const uint32_t key = order_key(x);
        if (cand && bin12(key) == bstar) {
            const uint32_t slot = atomicAdd(&count, 1u);
            if (slot < (uint32_t)kAdaSeg) seg[slot] = key & 0x7FFFFFFFu;
        }
    };
    const uint32_t lo = j_begin < sp ? (uint32_t)(sp - j_begin) : 0u;        // the part's first candidate
#pragma unroll
    for (int u = 0; u < KPT; ++u) {
        const uint32_t o = (uint32_t)(u * kAdaThreads + tid);
        hand_in(v[u], o >= lo && o < len);
    }
    // parts longer than that: the rest streams through registers
    for (uint32_t o0 = (uint32_t)(KPT * kAdaThreads); o0 < len; o0 += (uint32_t)(kAdaU * kAdaThreads)) {
        float x[kAdaU];
#pragma unroll
        for (int u = 0; u < kAdaU; ++u) {
            const uint32_t o = o0 + (uint32_t)(u * kAdaThreads + tid);
            x[u] = o < len ? sc[o] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kAdaU; ++u) {
            const uint32_t o = o0 + (uint32_t)(u * kAdaThreads + tid);
            hand_in(x[u], o >= lo && o < len);
        }
    }
}

// bits per refinement level so that H digit histograms fit kAdaDigWords
__device__ __forceinline__ int ada_level_bits(int H) {
    int bits = 6;
    while (bits > 1 && (H << bits) > kAdaDigWords) --bits;
    return bits;
}

struct AdaShared {
    uint32_t wave_tot[kAdaWaves];
    uint32_t digit, want;
    uint32_t total_in;                            // keys inside the cut bin, all heads
    uint32_t slow;
    unsigned long long over;                      // sum of the heads' keys above the bin beyond their safeguards
    uint32_t scratch[kListScratch];
};

__global__ __launch_bounds__(kAdaThreads) void ada_allot_kernel(
    AdaWorkspace ws, const float* __restrict__ scores, int64_t n, int H, int32_t sp, int32_t g, long long R,
    int32_t k, int32_t* __restrict__ budgets, int64_t* __restrict__ offsets, BlockInfo* __restrict__ block_info,
    int layers) {
    extern __shared__ __align__(16) uint32_t dyn[];
    __shared__ AdaShared sm;
    const int layer = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int B0 = ada_level_bits(H);
    uint32_t* dig = dyn;                           // [H << B] digit histograms, then suffix sums
    uint32_t* above = dyn + kAdaDigWords;          // [H] keys above the prefix decided so far
    uint32_t* inbin = above + kAdaMaxHeads;        // [H] keys inside the cut bin; later: keys equal to the threshold
    uint32_t* base = inbin + kAdaMaxHeads;         // [H + 1] start of a head's keys in the list; later: its first row
    uint32_t* list = base + kAdaMaxHeads + 8;      // [kAdaList][2] (key, head)
    const uint32_t bstar = ws.layer[layer].bin;
    // ---- the heads' counts, the places of their keys in the list (a thread per head) ----------------------
    const uint32_t my_above = tid < H ? ws.above[(size_t)layer * H + tid] : 0u;
    const uint32_t my_in = tid < H ? ws.inbin[(size_t)layer * H + tid] : 0u;
    if (tid == 0) { sm.slow = bstar >= (uint32_t)(kBins12 - 1) ? 1u : 0u; sm.over = 0; }
    if (tid < kListScratch) sm.scratch[tid] = 0;
    // A head whose safeguard ends inside the bin counts from there on only.  Usually there is none: heads
    // beyond their safeguard before the bin count all of its keys, the others none of them, and the threshold is the key
    // of one rank among the former's.
    const bool beyond = my_above >= (uint32_t)g;
    const bool by_rank = !__syncthreads_or(tid < H && !beyond && (unsigned long long)my_above + my_in > (unsigned long long)g);
    const uint32_t listed = by_rank && !beyond ? 0u : my_in;
    uint32_t incl = wave_inclusive(listed);        // (wraps only where some head is beyond its segment)
    if (lane == 63) sm.wave_tot[wave] = incl;
    if (tid < H && beyond) atomicAdd(&sm.over, (unsigned long long)(my_above - (uint32_t)g));
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += sm.wave_tot[w];
    if (tid < H) {
        above[tid] = my_above;
        inbin[tid] = listed;
        base[tid] = incl - listed;
        if (tid == H - 1) sm.total_in = incl;
        if (my_in > (uint32_t)kAdaSeg || incl > (uint32_t)kAdaList) sm.slow = 1u;
    }
    __syncthreads();
    const bool slow = sm.slow != 0;
    const uint32_t total_in = slow ? 0u : sm.total_in;
    if (!slow) {
        // gather the heads' segments into one list; threads are dealt to heads so that all
        // heads' loads are in flight together
        int per_head = kAdaThreads / H;             // H <= 1024
        if (per_head < 1) per_head = 1;
        const int h = tid / per_head, r = tid - h * per_head;
        if (h < H) {
            const uint32_t* seg = ws.seg + ((size_t)layer * H + h) * kAdaSeg;
            const uint32_t cnt = inbin[h], b0 = base[h];
            for (uint32_t i = r; i < cnt; i += per_head) {
                list[2 * (b0 + i)] = seg[i];
                list[2 * (b0 + i) + 1] = (uint32_t)h;
            }
        }
        __syncthreads();
    }

    // ---- the key of a rank among the listed --------------------------------------------------------
    int rem = bstar < (uint32_t)(kBins12 - 1) ? kBinShift : 31;
    uint32_t fixed = bstar < (uint32_t)(kBins12 - 1) ? bstar : 0u;
    const unsigned long long rank = (unsigned long long)R - sm.over;           // (R is not reached above the bin)
    if (!slow && by_rank && rank >= 1 && rank <= total_in) {
        uint32_t need;
        for (int h = tid; h < H; h += kAdaThreads) dig[h] = 0;
        fixed = threshold_on_list<kAdaThreads>(reinterpret_cast<const int32_t*>(list), total_in, bstar, (uint32_t)rank, sm.scratch, &sm.digit,
                                               &sm.want, &need);
        __syncthreads();
        for (uint32_t i = tid; i < total_in; i += kAdaThreads) {
            const uint32_t key = list[2 * i], h = list[2 * i + 1];
            if (key > fixed) atomicAdd(&above[h], 1u);
            else if (key == fixed) atomicAdd(&dig[h], 1u);
        }
        __syncthreads();
        for (int h = tid; h < H; h += kAdaThreads) inbin[h] = dig[h];
        rem = 0;
        __syncthreads();
    }
    // ---- or refined below the bin: B bits per level ---------------------------------------------------
    // A key takes part while bin12(key) == bstar and its bits above `rem` equal `fixed`.
    const float* lsc = scores + (size_t)layer * H * n;
    while (rem > 0) {
        const int B = rem < B0 ? rem : B0;
        const int D = 1 << B;
        const int shift = rem - B;
        for (int i = tid; i < (H << B); i += kAdaThreads) dig[i] = 0;
        __syncthreads();
        if (!slow) {
            for (uint32_t i = tid; i < total_in; i += kAdaThreads) {
                const uint32_t key = list[2 * i], h = list[2 * i + 1];
                if ((key >> rem) == fixed) atomicAdd(&dig[(h << B) | ((key >> shift) & (uint32_t)(D - 1))], 1u);
            }
        } else {
            for (int h = 0; h < H; ++h) {
                const float* hs = lsc + (size_t)h * n;
                for (int64_t j0 = tid; j0 < n; j0 += (int64_t)kAdaU * kAdaThreads) {
                    float v[kAdaU];
#pragma unroll
                    for (int u = 0; u < kAdaU; ++u) {
                        const int64_t j = j0 + (int64_t)u * kAdaThreads;
                        v[u] = j < n ? hs[j] : 0.f;
                    }
#pragma unroll
                    for (int u = 0; u < kAdaU; ++u) {
                        const int64_t j = j0 + (int64_t)u * kAdaThreads;
                        const uint32_t key = order_key(v[u]);
                        const uint32_t k31 = key & 0x7FFFFFFFu;
                        if (j >= sp && j < n && bin12(key) == bstar && (rem >= 31 || (k31 >> rem) == fixed))
                            atomicAdd(&dig[((uint32_t)h << B) | ((k31 >> shift) & (uint32_t)(D - 1))], 1u);
                    }
                }
            }
        }
        __syncthreads();
        // suffix sums per head: dig[h][d] = keys of head h in this prefix with digit >= d.  A wave
        // per head, lane L on digit D-1-L (D <= 64).
        for (int h = wave; h < H; h += kAdaWaves) {
            uint32_t incl = lane < D ? dig[(h << B) | (D - 1 - lane)] : 0u;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t t = __shfl_up(incl, off, 64);
                if (lane >= off) incl += t;
            }
            if (lane < D) dig[(h << B) | (D - 1 - lane)] = incl;
        }
        __syncthreads();
        if (wave == 0) {                            // lane d: does the sum reach R when digits >= d count?
            bool ok = false;
            if (lane < D) {
                unsigned long long e = 0;
                for (int h = 0; h < H; ++h) {
                    const uint32_t c = above[h] + dig[(h << B) | lane];
                    if (c > (uint32_t)g) e += c - (uint32_t)g;
                }
                ok = e >= (unsigned long long)R;
            }
            const unsigned long long m = __ballot(ok);
            if (lane == 0) sm.digit = m ? (uint32_t)(63 - __clzll((long long)m)) : 0u;   // the largest such digit
        }
        __syncthreads();
        const uint32_t digit = sm.digit;
        const bool last_level = shift == 0;
        for (int h = tid; h < H; h += kAdaThreads) {
            const uint32_t ge = dig[(h << B) | digit];
            const uint32_t gt = digit + 1 < (uint32_t)D ? dig[(h << B) | (digit + 1)] : 0u;
            above[h] += gt;
            if (last_level) inbin[h] = ge - gt;    // keys equal to the threshold
        }
        fixed = rem >= 31 ? digit : ((fixed << B) | digit);
        rem = shift;
        __syncthreads();
    }

    // ---- exact threshold reached: above[h] keys beat it, inbin[h] keys equal it -------------------
    if (H <= 64 && (long long)H * n <= 0x7FFFFFFFll) {
        if (wave == 0) {                            // a lane per head, what the loop below does
            const bool on = lane < H;
            const uint32_t cp = on ? above[lane] : 0u, eq = on ? inbin[lane] : 0u, ug = (uint32_t)g;
            const uint32_t over = on && cp > ug ? cp - ug : 0u;
            const long long total_over = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive(over), 63);
            const uint32_t rest = R > total_over ? (uint32_t)(R - total_over) : 0u;
            const uint32_t kept = cp > ug ? cp : ug;
            const uint32_t open_eq = on && cp + eq > kept ? cp + eq - kept : 0u;
            const uint32_t before = wave_inclusive(open_eq) - open_eq;
            const uint32_t left = rest > before ? rest - before : 0u;
            const uint32_t take = open_eq < left ? open_eq : left;
            uint32_t b = (uint32_t)sp + kept + take;
            b = !on ? 0u : b > (uint32_t)n ? (uint32_t)n : b;
            const uint32_t layer_rows = (uint32_t)H * (uint32_t)k;
            const uint32_t run = wave_inclusive(b) - b;
            if (on) {
                budgets[(size_t)layer * H + lane] = (int32_t)b;
                ws.known[(size_t)layer * H + lane] = Threshold{cp >= ug ? fixed : kNoThreshold, take};
                base[lane] = run < layer_rows ? run : layer_rows;
            }
            if (lane == 0) base[H] = layer_rows;
        }
    } else if (tid == 0) {
        int32_t* out = budgets + (size_t)layer * H;
        long long rest = R;
        for (int h = 0; h < H; ++h)
            if (above[h] > (uint32_t)g) rest -= (long long)(above[h] - (uint32_t)g);
        if (rest < 0) rest = 0;
        const long long layer_rows = (long long)H * k;
        long long run = 0;
        for (int h = 0; h < H; ++h) {
            const long long cp = above[h], eq = inbin[h];
            const long long kept = cp > g ? cp : g;             // before any tied key is allotted
            long long open_eq = cp + eq - kept;                  // tied keys the safeguard does not cover
            if (open_eq < 0) open_eq = 0;
            const long long take = open_eq < rest ? open_eq : rest;
            rest -= take;
            long long b = sp + kept + take;
            b = b > n ? n : b;
            out[h] = (int32_t)b;
            // a head that keeps more than its safeguard keeps exactly the keys above the layer's
            // threshold and `take` of those equal to it: the selection need not search
            Threshold th;
            th.key31 = cp >= g ? fixed : kNoThreshold;
            th.need = (uint32_t)take;
            ws.known[(size_t)layer * H + h] = th;
            base[h] = (uint32_t)run;                 // the head's first row inside the layer
            run += b;
            if (run > layer_rows) run = layer_rows;  // whatever the counts were, a layer stays inside its rows
        }
        base[H] = (uint32_t)layer_rows;
    }
    if (!offsets) return;
    __syncthreads();
    // ---- prefix sums and the gather's block table for this layer's rows ---------------------------
    const long long row0 = (long long)layer * H * k;
    for (int h = tid; h < H; h += kAdaThreads) offsets[(size_t)layer * H + h] = row0 + base[h];
    if (tid == 0 && layer == layers - 1) offsets[(size_t)layers * H] = row0 + base[H];
    const long long row1 = row0 + (long long)H * k;
    const long long b_first = (row0 + kCompactRowsPerBlock - 1) / kCompactRowsPerBlock;
    for (long long b = b_first + tid; b * kCompactRowsPerBlock < row1; b += kAdaThreads) {
        const uint32_t p = (uint32_t)(b * kCompactRowsPerBlock - row0);     // row inside the layer
        int lo = 0, hi = H - 1;                    // first head whose rows end beyond p (base[H] > p)
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (base[mid + 1] > p) hi = mid; else lo = mid + 1;
        }
        BlockInfo bi;
        bi.head_end = row0 + base[lo + 1];
        bi.head = layer * H + lo;
        bi.pad = 0;
        block_info[b] = bi;
    }
}

__global__ void ada_uniform_kernel(int32_t* __restrict__ budgets, int count, int32_t value) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) budgets[i] = value;
}

// ---- offsets and gather block table from budgets that only exist on the device -------------
// (for the cases in which nothing is allotted layer-wide and every head gets the same budget)
// One workgroup walks the heads in order, 1024 at a time.  Prefix sums are kept within
// [0, total] and the last offset is total, so that whatever the budgets hold, the selection
// and gather kernels that follow stay inside buffers sized for `total` rows.
__device__ __forceinline__ void ada_block_entry(const int64_t* offsets, int heads, int64_t b, BlockInfo* info);

__global__ __launch_bounds__(kAdaThreads) void ada_offsets_kernel(const int32_t* __restrict__ budgets, int heads,
                                                                  int64_t n, int64_t total,
                                                                  int64_t* offsets,      // written, then read back below
                                                                  int64_t blocks_here, BlockInfo* info) {
    __shared__ long long wave_tot[kAdaWaves];
    __shared__ long long carry_s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) { carry_s = 0; offsets[0] = 0; }
    __syncthreads();
    for (int base = 0; base < heads; base += kAdaThreads) {
        const int i = base + tid;
        long long b = i < heads ? (long long)budgets[i] : 0;
        b = b < 0 ? 0 : (b > n ? n : b);
        long long incl = b;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        if (lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        long long before = carry_s;
        for (int w = 0; w < wave; ++w) before += wave_tot[w];
        if (i < heads) {
            const long long end = before + incl;
            offsets[i + 1] = (i == heads - 1 || end > total) ? total : end;
        }
        __syncthreads();
        if (tid == kAdaThreads - 1) carry_s = before + incl;
        __syncthreads();
    }
    // a table of moderate size is filled right here (blocks_here = 0: a launch of its own does it)
    for (int64_t b = tid; b < blocks_here; b += kAdaThreads) ada_block_entry(offsets, heads, b, info);
}

// block b of the gather starts at row b*kCompactRowsPerBlock: the head owning that row is the
// first one whose rows end beyond it
__device__ __forceinline__ void ada_block_entry(const int64_t* offsets, int heads, int64_t b, BlockInfo* info) {
    const int64_t p = b * kCompactRowsPerBlock;
    int lo = 0, hi = heads - 1;                    // offsets[heads] = total > p, so the answer exists
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (offsets[mid + 1] > p) hi = mid; else lo = mid + 1;
    }
    BlockInfo bi;
    bi.head_end = offsets[lo + 1];
    bi.head = lo;
    bi.pad = 0;
    info[b] = bi;
}

__global__ void ada_blocks_kernel(const int64_t* __restrict__ offsets, int heads, int64_t blocks,
                                  BlockInfo* __restrict__ info) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b < blocks) ada_block_entry(offsets, heads, b, info);
}

hipError_t launch_adaptive_plan(const curdkv_ctx* ctx, const int32_t* budgets, int64_t n, int64_t total,
                                int64_t* offsets, BlockInfo* block_info, hipStream_t stream) {
    const int64_t blocks = (total + kCompactRowsPerBlock - 1) / kCompactRowsPerBlock;
    // a table of one entry per thread is filled by the offsets kernel itself; a longer one by a
    // launch of its own (one workgroup walking 6552 entries took 10 us, the extra launch 5)
    const bool small = blocks <= kAdaThreads;
    ada_offsets_kernel<<<dim3(1), kAdaThreads, 0, stream>>>(budgets, ctx->heads, n, total, offsets,
                                                           small ? blocks : 0, block_info);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || small) return e;
    ada_blocks_kernel<<<dim3((unsigned)((blocks + 255) / 256)), 256, 0, stream>>>(offsets, ctx->heads, blocks, block_info);
    return hipGetLastError();
}

// dynamic LDS of ada_allot_kernel: digit histograms, three per-head arrays and the key list
constexpr size_t kAdaAllotLds = ((size_t)kAdaDigWords + 3 * (size_t)kAdaMaxHeads + 8 + 2 * (size_t)kAdaList) * 4;

// The layout above holds for every head count the kernel accepts: digit histograms of at least
// one bit per level, and everything inside the 160 KB of a gfx950 workgroup beside the static
// part (AdaShared and the compiler's own few words).
static_assert((kAdaMaxHeads << 1) <= kAdaDigWords, "a level of one bit must fit the digit histograms");
static_assert(kAdaAllotLds + sizeof(AdaShared) + 1024 <= 160 * 1024, "ada_allot_kernel's LDS");
static_assert(kAdaSeg <= kAdaList, "one head's segment must fit the list");

hipError_t configure_adaptive(curdkv_ctx* ctx) {
    if ((size_t)ctx->lds_limit < kAdaAllotLds + 4096) return hipSuccess;    // the adaptive calls then report an error
    return hipFuncSetAttribute((const void*)ada_allot_kernel,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAdaAllotLds);
}

size_t adaptive_workspace_bytes(const curdkv_ctx* ctx) {
    return workspace_bytes_for(slots_for(ctx), (size_t)ctx->heads, (size_t)ctx->cfg.layers);
}

// ---- the same workspace as a static device array, for callers that cannot allocate ----------
// curdkv_adaptive_budgets_noalloc runs the kernels above on this array instead of a buffer
// from hipMalloc.  Every GPU the library is used on holds its own copy, at its own address,
// from the moment the code object is loaded until the process ends.  On the host the array's
// name is only a handle for hipGetSymbolAddress: the address the kernels are given is the one
// that call returns, looked up once per device at curdkv_create.  Nothing in the array has to
// hold a particular value when a call starts: the kernels set what they read.
constexpr int kScratchMaxHeads = 1024;                 // layers * kv_heads the static workspace covers
constexpr size_t kScratchBytes = workspace_bytes_for(kScratchMaxHeads, kScratchMaxHeads, kScratchMaxHeads);   // 24.5 MiB + 32 KiB
static_assert(kScratchMaxHeads >= kAdaSlots, "fewer heads than histograms take no more room");
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kScratchMaxDevices = 64;
static void* g_scratch_ptr[kScratchMaxDevices];        // device address of `scratch`, per device
static std::mutex g_scratch_mutex;

int adaptive_static_max_heads() { return kScratchMaxHeads; }

// Called with `device` current.  Looks the array's device address up on first use.
hipError_t adaptive_static_workspace_init(int device) {
    if (device < 0 || device >= kScratchMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[device]) return hipSuccess;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}

void* adaptive_static_workspace(int device) {
    if (device < 0 || device >= kScratchMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    return g_scratch_ptr[device];
}

uint32_t* adaptive_hist_buffer(const curdkv_ctx* ctx, void* workspace) {
    return carve(workspace, ctx).hist;
}

uint32_t* adaptive_coarse_buffer(const curdkv_ctx* ctx, void* workspace) {
    return carve(workspace, ctx).coarse;
}

const void* adaptive_thresholds(const curdkv_ctx* ctx, void* workspace) {
    return carve(workspace, ctx).known;
}

bool adaptive_allots(int32_t k, int32_t sp, long long R) { return k > sp && R > 0; }

hipError_t launch_adaptive(const curdkv_ctx* ctx, void* workspace, float* scores, int64_t n, int32_t k,
                           int32_t sp, int32_t g, long long R, int32_t* budgets, hipStream_t stream,
                           bool hist_ready, int scale_blocks, int64_t* offsets, BlockInfo* block_info, bool* planned) {
    const int H = ctx->cfg.kv_heads, L = ctx->cfg.layers;
    if (planned) *planned = false;
    if (!adaptive_allots(k, sp, R)) {           // nothing to allot: k each, or all covered by the safeguard
        const int32_t v = k <= sp ? k : sp + g;
        ada_uniform_kernel<<<dim3((unsigned)((ctx->heads + 255) / 256)), 256, 0, stream>>>(budgets, ctx->heads, v);
        return hipGetLastError();
    }
    if ((size_t)ctx->lds_limit < kAdaAllotLds + 4096 || H > kAdaMaxHeads) return hipErrorInvalidConfiguration;
    const AdaWorkspace ws = carve(workspace, ctx);
    const int parts = hist_ready ? 1 : parts_for(ctx->heads, n);
    const int64_t part = (n + parts - 1) / parts;
    const dim3 grid((unsigned)parts * (unsigned)ctx->heads);
    if (!hist_ready) ada_hist_kernel<<<grid, kAdaThreads, 0, stream>>>(scores, n, sp, parts, part, ws.hist, ws.coarse, ctx->d_partial, scale_blocks);
    auto cut = [&](auto kpt) {
        ada_cut_kernel<decltype(kpt)::value><<<grid, kAdaThreads, 0, stream>>>(ws, scores, n, H, sp, g, R, parts, part);
    };
    if (part <= 4 * kAdaThreads) cut(std::integral_constant<int, 4>{});
    else if (part <= 16 * kAdaThreads) cut(std::integral_constant<int, 16>{});
    else cut(std::integral_constant<int, kAdaOwn>{});
    // the kernel keeps a head's first row inside its layer in 32 bits: a layer of 2^32 rows or
    // more gets its offsets and block table from the general kernels instead
    if ((long long)H * k > 0xFFFFFFFFll) offsets = nullptr;
    ada_allot_kernel<<<dim3((unsigned)L), kAdaThreads, kAdaAllotLds, stream>>>(
        ws, scores, n, H, sp, g, R, k, budgets, offsets, offsets ? block_info : nullptr, L);
    if (planned) *planned = offsets != nullptr;
    return hipGetLastError();
}

}  // namespace curdkv
