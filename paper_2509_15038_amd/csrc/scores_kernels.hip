// Scoring kernels: the projection, row-norm-squared, combination and
// normalisation steps of Algorithm 1, for gfx950.
//
// One pass over K and V.  The projection is computed transposed,
//     Y^T = G^T A^T   (A = K_i or V_i),
// with G^T as the MFMA A operand (M = sketch columns) and a tile of token rows
// as the B operand (N = tokens).  In the accumulator layout a lane then owns
// several sketch coordinates of ONE token (its column), so the row-norm squared
// is a sum inside the lane plus one or two lane exchanges.  The projected rows
// never leave registers.  The bf16 inner loop lives in scan_device.h.

#include "scan_device.h"
#include "select_device.h"

namespace curdkv {

// Sum the wave totals of a block (four or eight) in a fixed order and store it.  A head
// scored by a single block (few new tokens during generation) can fold the total into the
// head's running sum right here: sum = (restart ? 0 : sum) + total, in double, which is
// what accumulate_few_kernel computes from one partial.
template <int WAVES>
__device__ __forceinline__ void block_partial_store(float wave_total, float* dst, double* running, int restart) {
    __shared__ float wsum[WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) wsum[wave] = wave_total;
    __syncthreads();
    if (threadIdx.x == 0) {
        float total = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
        if (WAVES == 8) total += (wsum[WAVES - 4] + wsum[WAVES - 3]) + (wsum[WAVES - 2] + wsum[WAVES - 1]);
        *dst = total;
        if (running) *running = (restart ? 0.0 : *running) + (double)total;
    }
}

// ---------------------------------------------------------------------------
// bf16 storage.  Each wave scores a contiguous range of tiles (scan_device.h),
// collecting the scores in its own slice of LDS, and writes them out in one
// burst per stage: no global store sits inside the streaming loop.  Score
// writes that mingle with the read streams of other waves are dear on this
// memory system (1 % of the bytes cost 7 % of the time with 8 KB stages), so the
// stages are as large as LDS allows, normally a wave's whole range: the workgroups of one round then
// end, and write, at about the same time.  The stores are ordinary ones, which leave the scores in the caches for the kernel
// that normalises or selects (non-temporal: curdkv_scores of 112 heads of 10007 tokens 94.3 us, so 92.5; one call for 32 of 32768 118.6 and 117.0).
// ---------------------------------------------------------------------------
template <int CB> struct Stage {    // tiles (of 32 tokens) a wave collects between bursts
    static constexpr int kTiles = CB > 4 ? 256 : 128;     // one workgroup per CU: 128 KB; two: 64 KB each
};

// COUNT: the workgroup also leaves its histogram of scores for the split selection (split_select.hip).
// MODE: rows past the caches or not (kStream* in scan_device.h).
template <int CB, int SRC, bool PROJ, bool COUNT, int MODE>
__global__ __launch_bounds__(256, (CB <= 4 ? 2 : 1)) void scores_bf16_kernel(
    const uint4* __restrict__ K, const uint4* __restrict__ V, const uint4* __restrict__ Gp,
    float* __restrict__ scores, float* __restrict__ partial, int64_t n, int blocks_per_head,
    int64_t out_stride, int64_t out_offset, double* __restrict__ sums, int restart,
    uint32_t* __restrict__ hist_out, uint32_t* __restrict__ coarse_out, int hists, int32_t n_sink, CachedShares share) {
    constexpr int kStageTiles = Stage<CB>::kTiles;
    __shared__ float stage[4][kStageTiles * kTileTokens];
    __shared__ uint32_t hist[COUNT ? kRawHistWords : 1];
    const int head = blockIdx.x / blocks_per_head;
    const int blk = blockIdx.x - head * blocks_per_head;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    if (COUNT) {                                   // (before any load goes out: the barrier would wait for it)
        for (int i = threadIdx.x; i < kRawHistWords; i += 256) hist[i] = 0;
        __syncthreads();
    }
    SketchRegs<CB> G;
    if (PROJ) load_sketch<CB>(G, Gp + (size_t)head * (CB * 4 * 64), lane);

    const int32_t n32 = (int32_t)n;
    const int32_t tiles = (n32 + kTileTokens - 1) / kTileTokens;
    const int32_t waves_per_head = blocks_per_head * 4;
    int32_t per_wave = (tiles + waves_per_head - 1) / waves_per_head;
    per_wave += per_wave & 1;                                   // whole pairs
    const int32_t t_begin = (blk * 4 + wave) * per_wave;
    const int32_t t_end = t_begin + per_wave < tiles ? t_begin + per_wave : tiles;
    const uint4* Kh = K + (size_t)head * n * 16;                // 16 chunks of 16 bytes per row
    const uint4* Vh = V + (size_t)head * n * 16;
    float* sh = scores + (size_t)head * out_stride + out_offset;   // score of row j goes to sh[j]
    float* mine = stage[wave];
    float acc_sum = 0.f;
    const CachedTiles cached = cached_tiles(t_begin, t_end, share);
    for (int32_t seg = t_begin; seg < t_end; seg += kStageTiles) {
        const int32_t seg_end = seg + kStageTiles < t_end ? seg + kStageTiles : t_end;
        const int32_t r0 = seg * kTileTokens;
        acc_sum += scan_tiles<CB, SRC, PROJ, COUNT, MODE>(G, Kh, Vh, n32, seg, seg_end, mine, r0, lane,
                                                   // (streamed rows gain nothing from different starts here: 32 heads of 32768 tokens 89.7 us with, 89.0 without, appends of
                                                   // 1024 tokens to 256 heads 24.5 and 23.5; the kernel of one workgroup a head does, 256 of 32768 623 and 630)
                                                   MODE == kStreamNone ? scan_phase(head, blk * 4 + wave) : 0u, hist, n_sink, cached);
        const int32_t r1 = seg_end * kTileTokens < n32 ? seg_end * kTileTokens : n32;
        for (int32_t r = r0 + lane; r < r1; r += 64) sh[r] = mine[r - r0];
    }
    block_partial_store<4>(wave_sum(acc_sum), partial + (size_t)head * kMaxBlocksPerHead + blk,
                           sums ? sums + head : nullptr, restart);
    if (COUNT) raw_hist_store<256>(hist, hist_out, coarse_out, head * hists + blk);
}

// ---------------------------------------------------------------------------
// fp32 storage: the same structure (scan_device.h).  CB = 16-column blocks of the padded sketch.
// SPLIT: the products go over the bf16 matrix units; the sketch's parts share the LDS with the score stages, and a workgroup has eight waves,
// two to a SIMD.  Otherwise (CB = 2: up to 32 columns, and the ablation without projection) the sketch is in registers and a
// lane's two tile buffers take 256 more: a SIMD holds one wave and a compute unit one workgroup of four.
// STREAM: rows past the caches, as above.
// ---------------------------------------------------------------------------
template <int CB, bool SPLIT> struct ShapeF32 {
    static constexpr int kWaves = SPLIT ? 8 : 4;
    static constexpr int kTiles = CB > 4 ? 48 : CB > 2 ? 96 : SPLIT ? 112 : 256;    // per wave between bursts: 48, 96, 112 or 128 KB in all
};

template <int CB, int SRC, bool PROJ, bool COUNT, bool SPLIT, bool STREAM>
__global__ __launch_bounds__((ShapeF32<CB, SPLIT>::kWaves * 64), (SPLIT ? 2 : 1)) void scores_f32_kernel(
    const float4* __restrict__ K, const float4* __restrict__ V, const float4* __restrict__ Gp,
    float* __restrict__ scores, float* __restrict__ partial, int64_t n, int blocks_per_head,
    int64_t out_stride, int64_t out_offset, double* __restrict__ sums, int restart,
    uint32_t* __restrict__ hist_out, uint32_t* __restrict__ coarse_out, int hists, int32_t n_sink, CachedShares share) {
    constexpr int kWaves = ShapeF32<CB, SPLIT>::kWaves;
    constexpr int kStageTiles = ShapeF32<CB, SPLIT>::kTiles;
    __shared__ float stage[kWaves][kStageTiles * kTileTokens];
    __shared__ bf16x8 gs[SPLIT ? kSketchF32Chunks<CB> : 1];
    __shared__ uint32_t hist[COUNT ? kRawHistWords : 1];
    const int head = blockIdx.x / blocks_per_head;
    const int blk = blockIdx.x - head * blocks_per_head;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    if (COUNT) {
        for (int i = threadIdx.x; i < kRawHistWords; i += kWaves * 64) hist[i] = 0;
        __syncthreads();
    }
    const float4* Gh = Gp + (size_t)head * (CB * 8 * 64);
    SketchF32<SPLIT ? 1 : CB> G;
    if constexpr (SPLIT) {
        split_sketch_to_lds<CB, kWaves * 64>(gs, Gh);
    } else if constexpr (PROJ) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int s = 0; s < 8; ++s) G.g[cb][s] = Gh[(cb * 8 + s) * 64 + lane];
    }

    const int32_t n32 = (int32_t)n;
    const int32_t tiles = (n32 + kTileTokens - 1) / kTileTokens;
    const int32_t waves_per_head = blocks_per_head * kWaves;
    int32_t per_wave = (tiles + waves_per_head - 1) / waves_per_head;
    per_wave += per_wave & 1;                                   // whole pairs
    const int32_t t_begin = (blk * kWaves + wave) * per_wave;
    const int32_t t_end = t_begin + per_wave < tiles ? t_begin + per_wave : tiles;
    const float4* Kh = K + (size_t)head * n * 32;               // 32 chunks of 16 bytes per row
    const float4* Vh = V + (size_t)head * n * 32;
    float* sh = scores + (size_t)head * out_stride + out_offset;
    float* mine = stage[wave];
    float acc_sum = 0.f;
    const CachedTiles cached = cached_tiles(t_begin, t_end, share);
    for (int32_t seg = t_begin; seg < t_end; seg += kStageTiles) {
        const int32_t seg_end = seg + kStageTiles < t_end ? seg + kStageTiles : t_end;
        const int32_t r0 = seg * kTileTokens;
        const uint32_t phase = scan_phase(head, blk * kWaves + wave);
        if constexpr (SPLIT) acc_sum += scan_tiles_f32_split<CB, SRC, COUNT, STREAM>(gs, Kh, Vh, n32, seg, seg_end, mine, r0, lane, phase, hist, n_sink, cached);
        else acc_sum += scan_tiles_f32<CB, SRC, PROJ, COUNT>(G, Kh, Vh, n32, seg, seg_end, mine, r0, lane, phase, hist, n_sink);
        const int32_t r1 = seg_end * kTileTokens < n32 ? seg_end * kTileTokens : n32;
        for (int32_t r = r0 + lane; r < r1; r += 64) sh[r] = mine[r - r0];
    }
    block_partial_store<kWaves>(wave_sum(acc_sum), partial + (size_t)head * kMaxBlocksPerHead + blk,
                                sums ? sums + head : nullptr, restart);
    if (COUNT) raw_hist_store<kWaves * 64>(hist, hist_out, coarse_out, head * hists + blk);
}

// Few tokens in all (scan_few): `steps` of 16 tokens to a workgroup.
template <bool F32, int CB, int SRC>
__global__ __launch_bounds__(((SRC == kSrcKV ? 2 : 1) * CB * 64)) void scores_few_kernel(
    const typename FewOperand<F32>::Word* __restrict__ K, const typename FewOperand<F32>::Word* __restrict__ V,
    const typename FewOperand<F32>::Word* __restrict__ Gp, float* __restrict__ scores, float* __restrict__ partial, int32_t n,
    int32_t blocks_per_head, int32_t steps, int64_t out_stride, int64_t out_offset, double* __restrict__ sums, int restart) {
    constexpr int kRow = 4 * FewOperand<F32>::kSteps;           // 16-byte words per row
    __shared__ float red[2][(SRC == kSrcKV ? 2 : 1) * CB][16];
    const int head = blockIdx.x / blocks_per_head;
    const int blk = blockIdx.x - head * blocks_per_head;
    const int32_t all = (n + 15) / 16;
    const int32_t first = blk * steps < all ? blk * steps : all;
    const int32_t last = first + steps < all ? first + steps : all;
    float* sh = scores + (size_t)head * out_stride + out_offset;
    float acc = 0.f;
    scan_few<F32, CB, SRC>(Gp + (size_t)head * (CB * FewOperand<F32>::kSteps * 64), K + (size_t)head * n * kRow,
                           V + (size_t)head * n * kRow, n, first, last, red, [&](int32_t row, float score) {
                               sh[row] = score;
                               acc += score;
                           });
    if (threadIdx.x < 64) {
        const float total = wave_sum(acc);
        if (threadIdx.x == 0) {
            partial[(size_t)head * kMaxBlocksPerHead + blk] = total;
            if (sums) sums[head] = (restart ? 0.0 : sums[head]) + (double)total;
        }
    }
}

// ---------------------------------------------------------------------------
// Normalisation step of Algorithm 1: divide by the sum over all n rows of the head.  The per-block
// partial sums are added in a fixed order in double, so the result does not
// depend on scheduling.  A zero sum gives 1/n everywhere.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void normalise_kernel(float* __restrict__ scores,
                                                        const float* __restrict__ partial,
                                                        int64_t n, int blocks_per_head,
                                                        int chunks_per_head) {
    const int head = blockIdx.x / chunks_per_head;
    const int chunk = blockIdx.x - head * chunks_per_head;
    partial += (size_t)head * kMaxBlocksPerHead;
    // one or two sums (many heads) come through scalar loads: 256 heads of 131072 tokens 42 us, 57 with all lanes adding
    const HeadScale scale = blocks_per_head <= 2
        ? scale_by((double)partial[0] + (blocks_per_head == 2 ? (double)partial[1] : 0.0), n)
        : head_scale(head_partial(partial, blocks_per_head), blocks_per_head, n);
    float* sh = scores + (size_t)head * n;
    constexpr int kInFlight = 8;                   // loads issued before the first store
    const int64_t stride = (int64_t)chunks_per_head * blockDim.x;
    for (int64_t j0 = (int64_t)chunk * blockDim.x + threadIdx.x; j0 < n; j0 += kInFlight * stride) {
        float v[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int64_t j = j0 + u * stride;
            v[u] = j < n ? sh[j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int64_t j = j0 + u * stride;
            if (j < n) sh[j] = scale(v[u]);
        }
    }
}

// GQA fold: mean over the query heads of a group.  The sum is taken in double,
// where adding a handful of floats is exact, so equal inputs come back unchanged.
__global__ __launch_bounds__(256) void fold_kernel(const float* __restrict__ sq,
                                                   float* __restrict__ out, int64_t n, int group,
                                                   int chunks_per_head) {
    const int head = blockIdx.x / chunks_per_head;
    const int chunk = blockIdx.x - head * chunks_per_head;
    const float* src = sq + (size_t)head * group * n;
    float* dst = out + (size_t)head * n;
    for (int64_t j = (int64_t)chunk * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)chunks_per_head * blockDim.x) {
        double s = 0.0;
        for (int q = 0; q < group; ++q) s += (double)src[(size_t)q * n + j];
        dst[j] = (float)(s / (double)group);
    }
}

// Products of up to 32 columns of an fp32 cache: over the bf16 units, rows past the caches, where every wave of the chip has 64 tokens or more
// (eight waves a compute unit) and the waves' shares, whole groups of 64, differ little, else in fp32.  There HBM waits for neither the matrix units nor the splitting, while the fp32 units are busy 55 %
// of the time and one wave a SIMD does not hide the rest.  curdkv_scores, r = 20, us, fp32 units and split: 8 heads of 4096 tokens 19.0 and 25.0, of 8192 22.7 and
// 25.5, of 16384 (64 tokens a wave) 35.6 and 31.9, of 20000 (64 or 128) 41.1 and 41.5, of 24000 45.7 and 43.5, of 32768 60.5 and 59.2, of 65536 106.4 and 95.5; 64 of 16384 198.9 and 178.1; 112 of
// 10007 211.2 and 197.2; 256 of 512 35.5 and 31.8, of 16384 727 and 685.  A sketch of the caller's that the split parts do not hold (sketch_splits) stays
// with the fp32 units.  Wider sketches are bound by the matrix units' power: streaming gives them
// nothing (64 heads of 16384, r = 64, 222.4 and 221.1).
static bool f32_split(const curdkv_ctx* ctx, int64_t n) {
    if (ctx->cfg.dtype != CURDKV_DTYPE_F32 || ctx->cfg.no_projection) return false;
    if (ctx->col_blocks > 1) return true;
    if (ctx->sketches_outside > 0) return false;
    const int64_t waves = (int64_t)ctx->num_cu * ShapeF32<2, true>::kWaves;
    if (ctx->heads * n < waves * 64) return false;
    const int64_t groups = (n + 63) / 64, places = waves / ctx->heads > 1 ? waves / ctx->heads : 1;
    return groups * 10 >= (groups + places - 1) / places * places * 7;
}

// Workgroups per head.  A workgroup should be long-lived (its start-up and the pipeline fill
// are paid per workgroup) and write its scores once, at its end, so the lower bound is what
// makes a wave's share fit its LDS stage.  Above that, the smallest count is taken that fills
// the rounds in which the workgroups pass through the chip to within 3 % of the best
// (measured at n = 32768: 4 per head for 384 heads, 7-8 for 288).  With no more heads than
// compute units the busiest unit decides: workgroups are dealt round-robin, so the cost is
// the number of workgroups a unit gets times their length, and ties go to the fewer, longer
// ones (measured at n = 32768, scoring and normalisation: 32 heads 8 per head, 64 heads 4,
// 128 heads 2; 2 to 5 % faster than filling two workgroups per unit).
// One exception, with the two-per-unit kernel: where one workgroup per head already puts four waves on three
// quarters of the compute units (192 or 224 heads of 256, or 448 of 512 places), HBM is saturated by those alone, and one long-lived workgroup per
// head, writing its scores in two bursts at most, beats any split although units stay idle. curdkv_scores, us, one and several per head: 192 heads of 4096 tokens 68.8 and 71.6, of 16384 246.8
// and 264.1, of 32768 527.5 and 523.2; 208 259.7 and 291.8, 553.6 and 602.1; 224 77.8 and 82.4, 276.5 and 326.3, 596.3 and 616.7; 448 of 8192 297.7 and 319.6, of 32768 1215 and 1258.
// Scans whose start would go through the caches (cached_shares) take it from four fifths on, below 257 heads: one call, a tenth kept, in turn, just written, behind other writes, 192 heads of 20000 tokens 425,
// 478, 446 and 402, 429, 408, of 32768 667, 755, 677 and 654, 695, 669, 200 689, 766, 697 and 684, 720, 696, 208 703, 787, 712 and 746, 789, 768, 224 751, 836, 764 and 769, 827, 797, 448 1490, 1574,
// 1511 and 1530, 1640, 1596.
static int pick_blocks_per_head(const curdkv_ctx* ctx, int64_t n, bool streams, int64_t most_blocks = kMaxBlocksPerHead) {
    const int64_t tiles = (n + kTileTokens - 1) / kTileTokens;
    const bool wide = ctx->cfg.dtype == CURDKV_DTYPE_BF16 && ctx->col_blocks > 2 && !ctx->cfg.no_projection;
    const bool f32 = ctx->cfg.dtype == CURDKV_DTYPE_F32;         // one workgroup per compute unit, like the wide kernel
    const int cb = ctx->cfg.no_projection ? 1 : ctx->col_blocks;
    const bool split = f32_split(ctx, n);
    const int waves = split ? ShapeF32<4, true>::kWaves : 4;         // per workgroup
    const int64_t stage = f32 ? (cb == 1 ? (split ? ShapeF32<2, true>::kTiles : ShapeF32<2, false>::kTiles) : cb == 2 ? ShapeF32<4, true>::kTiles : ShapeF32<8, true>::kTiles)
                              : (wide ? Stage<8>::kTiles : Stage<4>::kTiles);
    int64_t slots = (int64_t)ctx->num_cu * ((wide || f32 || ctx->heads <= ctx->num_cu) ? 1 : 2);
    // Few, long heads: a sixteenth of the units is left idle, and the ranges of the waves, which otherwise lie
    // powers of two apart where n is one, fall between.  Scoring, us with all 256 units and with 240 at most:
    // 8 heads of 131072 tokens 97.7 and 94.2, of 65536 51.5 and 49.9, of 32768 29.7 and 28.6, of 100000 74.1 and 73.6; 4 heads
    // of 131072 51.4 and 49.3; 16 of 32768 52.0 and 49.6; 32 of 32768 96.4 and 95.6, not worth a rule; 128 columns, 8 heads
    // of 131072 104.3 and 97.5.  Below eight tiles a wave the rounding to whole pairs costs more (8 heads of 8192:
    // 11.2 and 13.1).
    // Rows streamed past the caches (fetch in scan_device.h): 32 heads of 32768 tokens 89.1 and 86.8 as well, r = 20, 8 of 131072 85.7 and 83.5; but not with 128
    // columns, where every unit's matrix time counts (8 of 131072 91.0 and 93.8).
    const bool spare = ctx->cfg.dtype == CURDKV_DTYPE_BF16 && (streams ? !wide && ctx->heads * 8 <= ctx->num_cu : ctx->heads * 16 <= ctx->num_cu) &&
                       (int64_t)ctx->heads * tiles >= 8 * waves * slots;
    if (spare) slots -= slots / 16;
    int64_t cap = (tiles + waves - 1) / waves;                                     // at least one tile per wave
    if (cap > most_blocks) cap = most_blocks;
    int64_t lo = (tiles + waves * stage - 1) / (waves * stage);
    if (lo > cap) lo = cap;
    if (lo < 1) lo = 1;
    if (!wide && !f32 && lo <= 2 && ctx->heads <= 2 * (int64_t)ctx->num_cu) {
        const int64_t in_last = ctx->heads - (ctx->heads > ctx->num_cu ? ctx->num_cu : 0);   // heads in the last round
        const bool later = ctx->heads <= ctx->num_cu && cached_shares(ctx, n, 0, true).start > 0;
        if (later ? in_last * 5 >= 4 * (int64_t)ctx->num_cu : in_last * 4 >= 3 * (int64_t)ctx->num_cu) return 1;
    }
    // (up to one workgroup per place where the heads are few: 8 heads of 131072 tokens 105 us on 184 units, 99 on 256;
    // curdkv_scores of 1 head of 131072 tokens 34.6 us with 64 workgroups, 18.3 with 256, in fp32 77.1 and 36.8)
    const int64_t fill = (slots + ctx->heads - 1) / ctx->heads;
    const int64_t most = lo + 15 > fill ? lo + 15 : fill;
    int64_t hi = most < cap ? most : cap;
    if (spare && hi > slots / ctx->heads) hi = slots / ctx->heads > lo ? slots / ctx->heads : lo;     // one round
    auto cost = [&](int64_t b) {                                       // rounds x tiles a wave works through
        const int64_t rounds = ((int64_t)ctx->heads * b + slots - 1) / slots;
        int64_t per_wave = (tiles + waves * b - 1) / (waves * b);
        per_wave += per_wave & 1;                                      // whole pairs, as in the kernel
        return rounds * per_wave;
    };
    int64_t best = cost(lo);
    for (int64_t b = lo + 1; b <= hi; ++b) best = cost(b) < best ? cost(b) : best;
    for (int64_t b = lo; b <= hi; ++b)
        if (cost(b) * 100 <= best * 103) return (int)b;
    return (int)lo;
}

// As many workgroups as the chip holds at once (16 waves per compute unit), a step each at least: one more per head
// and some wait for a place (12 heads of 576 tokens, bf16, r = 128, 22 workgroups each 11.3 us per curdkv_scores_append, 21
// each 7.8).  Two steps stay in one workgroup in bf16, and in fp32 where a running sum is wanted, which it then adds by
// itself: one launch instead of two.  More than 64 a head, whose partial sums are then several to a lane, only for one or two
// heads, and while each has a compute unit to itself: two on a unit share its matrix units.  Replayed graph, us per
// curdkv_scores_append, up to 64 a head, up to one a unit, up to 256 a head: fp32, r = 64, 1 head of 8192 tokens 23.0, 9.2, 9.2; 2 heads of 6000 15.7,
// 10.7, 13.3; 3 of 3000 10.1, 10.1, 12.6; 3 of 4096 12.1, 12.6, 12.8; bf16, r = 20, 2 heads of 4096 5.4, 4.9, 5.3; 3 of 2048 4.8, 5.0, 5.2.
static int few_blocks_per_head(const curdkv_ctx* ctx, int64_t n, bool running) {
    const int waves = (ctx->cfg.score_source == CURDKV_SCORE_KV ? 2 : 1) * 2 * ctx->col_blocks;
    const int64_t slots = (int64_t)ctx->num_cu * (16 / waves);
    const int64_t steps = (n + 15) / 16;
    if (steps <= 2 && (running || ctx->cfg.dtype == CURDKV_DTYPE_BF16)) return 1;
    int64_t b = slots / ctx->heads;
    b = b < 1 ? 1 : b < steps ? b : steps;
    const int64_t units = ctx->num_cu / ctx->heads, most = ctx->heads > 2 || units < 64 ? 64 : units < kMaxBlocksPerHead ? units : kMaxBlocksPerHead;
    return (int)(b < most ? b : most);
}

// Calls of few tokens in all take scan_few.  Measured, us per curdkv_scores_append, the other kernel -> this one.
// fp32, r = 20 / 64 / 128: 16384 tokens in 8 heads 17.9 -> 12.1 / 23.8 -> 16.4 / 34.9 -> 21.6, 32768 tokens in 8
// heads 18.4 -> 16.1 / 24.7 -> 24.1 / 36.5 -> 36.4; in 256 heads level at 16384 tokens (13.2 -> 13.2 at
// r = 64) and behind at 32768 (15.3 -> 23.4).  Many steps in a workgroup cost more than they save (one head in 64 workgroups: 4096
// tokens, 4 steps each, 18.0 -> 11.3 / 23.8 -> 15.5 / 34.7 -> 23.2; 16384 tokens, 16 steps each,
// 20.7 -> 22.1 / 25.3 -> 36.2 / 36.2 -> 64.6).
// bf16: 256 heads of one token 4.4 -> 2.8 / 4.7 -> 3.1 / 5.5 -> 3.6; 8192 tokens in 8 heads 7.9 -> 5.1 / 8.6 -> 6.2 / 10.4 -> 8.0;
// 16384 in 8 heads 8.2 -> 5.9 / 9.0 -> 7.9 / 10.6 -> 11.4 and in 64 heads 6.6 -> 6.4 / 7.3 -> 8.1 / 9.0 -> 11.5; one head
// of 4096 tokens 8.6 -> 5.5 / 9.3 -> 7.4 / 11.1 -> 11.1.  Wide sketches in many heads end earlier, as each row goes to more
// waves: curdkv_scores, r = 64, 100 heads of 64 tokens 6.3 -> 6.7, 128 columns, 256 heads of 16 4.6 -> 4.8.
constexpr int64_t kFewF32Tokens = 16384, kFewF32Steps = 6, kFewBf16Tokens = 8192, kFewBf16Steps = 4;

// More tokens take it as long as the steps of a workgroup times the workgroups of a compute unit, which work one after the other, are few,
// by storage and sketch width, and the heads not so many that the other kernel fills the chip with one workgroup each.  One call, a fifth kept, us, the other
// kernel and this one (load): bf16, r = 20, 16 heads of 1024 tokens 13.6 and 11.6 (4), 8 of 3000 14.7 and 13.3 (6), 4 of 6000 15.6 and 14.9 (6), 3 of 8000 15.9 and
// 16.2 (8), 100 of 240 12.7 and 13.0 (8), 128 of 128 10.6 and 11.0 (4); r = 64, 8 of 2048 14.4 and 13.6 (4), 12 of 1300 14.3 and 13.6 (4), 24 of 680 14.0 and
// 15.0 (6), 48 of 200 12.3 and 13.0 (4); r = 128, 8 of 1200 15.2 and 14.8 (3), of 1600 15.6 and 16.9 (4).  fp32, r = 20, 8 of 4096 24.3 and 19.0 (8), 4 of 9000
// 26.4 and 23.0 (9), 256 of 128 23.2 and 21.4 (8), 16 of 3000 25.0 and 24.5 (12).  curdkv_scores_append: bf16, r = 20, 8 of 2048 8.5 and 7.1, r = 64 9.0 and
// 8.1; fp32, r = 20, 8 of 2500 18.3 and 11.0.  Wider fp32 sketches would gain as much (r = 64, 8 of 2500 30.2 and 23.4), but the split products of the other kernel err
// less than the plain ones here.
// fp32 in more heads than half the units: where one tensor is scored, or a running sum is wanted, the other kernel's one workgroup a head ends sooner (and adds
// the sum by itself): curdkv_scores_append, r = 20, 256 heads of 128 tokens, keys alone 8.2 and 12.4, 224 of 128 7.9 and 11.3, 200 of 160 8.6 and 11.1, both tensors 256 of 65
// 11.6 and 13.6, 224 of 128 12.6 and 13.6; curdkv_scores, keys alone, 256 of 128 10.6 and 12.9, 200 of 160 10.3 and 11.5, but both tensors 16.4 and 14.5, 16.8 and 14.4; up to
// 128 heads this one is ahead either way (128 of 160, keys alone, 8.5 and 7.0).
constexpr int kFewHeadsBf16 = 64, kFewLoadBf16 = 6;              // up to 32 columns
constexpr int kFewHeadsBf16Mid = 32, kFewLoadBf16Mid = 4;        // up to 64
constexpr int kFewHeadsBf16Wide = 32, kFewLoadBf16Wide = 3;      // up to 128
constexpr int kFewHeadsF32 = 256, kFewLoadF32 = 10;              // up to 32 columns

static bool few_by_load(const curdkv_ctx* ctx, int64_t load, bool running) {
    if (ctx->cfg.dtype == CURDKV_DTYPE_F32) {
        if (ctx->col_blocks > 1 || load > kFewLoadF32) return false;
        const bool one_less = running || ctx->cfg.score_source != CURDKV_SCORE_KV;
        return ctx->heads <= (one_less ? ctx->num_cu / 2 : kFewHeadsF32);
    }
    if (ctx->col_blocks == 1) return ctx->heads <= kFewHeadsBf16 && load <= kFewLoadBf16;
    if (ctx->col_blocks == 2) return ctx->heads <= kFewHeadsBf16Mid && load <= kFewLoadBf16Mid;
    return ctx->heads <= kFewHeadsBf16Wide && load <= kFewLoadBf16Wide;
}

// running: a running sum is wanted (curdkv_scores_append).
static bool few_tokens(const curdkv_ctx* ctx, int64_t n, bool running) {
    if (ctx->cfg.no_projection) return false;
    const bool f32 = ctx->cfg.dtype == CURDKV_DTYPE_F32;
    const int64_t most = f32 ? kFewF32Tokens : kFewBf16Tokens / (ctx->heads > ctx->num_cu / 4 ? ctx->col_blocks : 1);
    const int64_t steps = (n + 15) / 16, blocks = few_blocks_per_head(ctx, n, running);
    if (n * ctx->heads > most || steps > (f32 ? kFewF32Steps : kFewBf16Steps) * blocks) {
        const int64_t load = (steps + blocks - 1) / blocks * ((blocks * ctx->heads + ctx->num_cu - 1) / ctx->num_cu);
        if (!few_by_load(ctx, load, running)) return false;
    }
    // bf16, two steps of a wide sketch: the other kernel's waves hold all of it and take 32 tokens at once.  8 heads, r = 20 /
    // 64 / 128, replayed graph: 32 tokens 3.6 -> 3.4 / 3.9 -> 4.3 / 4.7 -> 6.3, 16 tokens 3.5 -> 3.0 / 3.8 -> 3.5 / 4.5 -> 4.6, 8
    // tokens 4.4 -> 3.9 at r = 128; curdkv_scores of 224 heads of 19 tokens, r = 64, in two workgroups 6.2 -> 6.8.
    const int64_t one_step = 32 / ctx->col_blocks;
    if (!f32 && n > one_step && n <= 32) return false;
    // bf16 appends that the other kernel gives one workgroup per head (up to 256 tokens) are one launch there, several
    // workgroups take a second one for the sum: 8 heads of 64 tokens 4.2 -> 4.5 / 4.7 -> 5.0 / 6.0 -> 6.0 replayed, 5.2 ->
    // 8.2 / 5.2 -> 8.4 / 6.1 -> 7.8 launched call by call, 8 heads of 256 6.6 -> 4.6 / 7.3 -> 5.1 / 8.9 -> 6.2 and
    // 6.7 -> 8.2 / 7.4 -> 8.5 / 9.0 -> 7.9: with 128 columns beyond 192 tokens the split wins either way (48 heads of 130
    // tokens 7.3 -> 7.9 and 7.7 -> 8.1).
    if (!f32 && running && n > 32 && !(ctx->col_blocks > 2 && n > 192) && pick_blocks_per_head(ctx, n, false) == 1) return false;
    return true;
}

// Whether rows are fetched past the caches (fetch in scan_device.h).  What fits the 256 MB Infinity Cache is often there already, and a gather
// of the same call finds its rows there.  us, kept in the caches and streamed, three caches in turn, r = 64: curdkv_scores of 8 heads of
// 24576 tokens (101 MB) 22.2 and 23.2, of 32768 (134) 31.2 and 29.0, of 65536 53.8 and 47.8; appends of 768 tokens to 256 heads (101) 19.8 and
// 20.6, of 1024 28.7 and 26.9; one call, a tenth kept, 8 heads of 8192 17.3 and 19.2, of 32768 (134) 44.8 and 45.4, of 40960 (168) 57.7 and 54.7, half
// kept (168, the end of the scan left in the caches) 75.9 and 78.6, 32 heads of 12288 (201) 81.6 and 79.1, 4 of 99162 (203) 88.2 and 95.7, 8 of 65536 (268) 110.6 and
// 108.3.  Large: 256 heads of 32768 703 and 624, of 131072, r = 128,
// 2858 and 2578.
constexpr int64_t kStreamBytes = 120000000, kStreamBytesReread = 160000000, kStreamBytesRereadMany = 256000000;
// Where a quarter of the rows or more are gathered afterwards, the end of the scan still goes through the caches: so much of it as
// the gather then finds there.  One call, half kept, nothing left, 128, 192 and 256 MB, us: 32 heads of 16384, r = 64, 103.9, 100.4, 109.0 and 110.7 (all
// kept in the caches 105.7); 256 of 32768 1326, 1304, 1309, 1311; fp32, r = 32, 8 heads of 32768 120.3, 109.7, 110.5, 113.0 (all 111.8), three tenths kept 101.2,
// 93.5, 94.4, 95.8 (95.3); in bf16 three tenths are level (32 of 16384 87.5 and 87.4).
constexpr int64_t kStayBytes = 128000000;

int64_t scan_bytes(const curdkv_ctx* ctx, int64_t n) {
    return ctx->heads * n * kHeadDim * (ctx->cfg.dtype == CURDKV_DTYPE_BF16 ? 2 : 4) * (ctx->cfg.score_source == CURDKV_SCORE_KV ? 2 : 1);
}

bool many_kept(const curdkv_ctx* ctx, int64_t n, int64_t kept) { return kept * 4 >= ctx->heads * n; }

// Where select_gather_kernel gathers uneven budgets, its workgroups that copy the large one's rows wait longer for those that come from HBM: from 256 MB on.  One call, 20 % kept, caches and streamed, Dirichlet budgets within layers of 8: 112 heads
// of 3487 tokens (200 MB) 68.0 and 74.6, 32 of 12207 74.1 and 77.4, 64 of 6103 in turn with writing them 136.7 and 146.9; one head of 8 with nearly all rows: 64 of 6103 68.9 and 76.2, of 7812
// (256 MB) 86.6 and 95.7, 32 of 17700 (290 MB) 104.3 and 110.6 (240 MB and more behind 270 MB of other traffic are ahead streamed, Dirichlet budgets: 32 of 14648 106.9 and 93.2).
// fp32 over the bf16 units: past the caches by any size for scores alone (r = 20, 8 heads of 16384 tokens, three in turn, 34.9 and 35.4, behind other writes 45.7 and 35.8; keys alone 22.2 and 21.2); a call that
// gathers from 256 MB on, whatever its budgets: 20 % kept, 8 of 24000 (197 MB), one cache again, in turn, behind reads, 64.3 and 70.3, 68.3 and 72.4, 68.4 and 73.9 (fp32 units, caches, 67, 70 and 70.5), just written 77.5 and 74.0, behind other writes
// 84.5 and 73.2; 32 of 4096 43.4 and 48.0, 46.5 and 48.8, 47.1 and 51.0; 200 of 1000 61 and 67, 67.9 and 68, 68.9 and 70.4; a tenth kept, 8 of 16384 42.3 and 46.3, 45.9 and 47.6, 47.1 and 48.8, keys alone 33.1
// and 31.9, 35.2 and 34.1, 35.6 and 35.4, of 32768 54.2 and 58.0, 60.3 and 60.2, 60.8 and 61.1; 268 MB, 8 of 32768, 76 and 82, 84 and 85, 85 and 86, behind other writes 105 and 85.
static bool stream_rows(const curdkv_ctx* ctx, int64_t n, int64_t kept, bool uneven) {
    const int64_t bytes = scan_bytes(ctx, n);
    if (ctx->cfg.dtype == CURDKV_DTYPE_F32) return ctx->col_blocks == 1 && f32_split(ctx, n) && (kept == 0 || bytes > kStreamBytesRereadMany);
    return bytes > (many_kept(ctx, n, kept) || uneven ? kStreamBytesRereadMany : kept > 0 ? kStreamBytesReread : kStreamBytes);
}

// What the kernel before has just written lies dirty in the Infinity Cache, and every non-temporal read of such a line writes it back. Where one workgroup takes long over a head
// those writes trickle in among the reads of the whole scan; rows read by ordinary loads at its start push the lines out at once (e^-(bytes / 256 MB) of them are left: it does not
// evict the oldest). One call, a tenth kept, K and V written just before: us, all through the caches, streamed, and streamed after 800 MB: 256 heads of 32768 tokens 909, 995 and
// 863, of 20000 592, 609 and 575, 224 of 32768 830, 853 and 828, 448 1601, 1667 and 1594, r = 128 256 934, 972 and 950, fp32, r = 20, of 24576 1352, 1443 and 1269. With other caches read before, 256 of 32768 take
// 848, 782 and 785, between calls of the same kind 856, 781 and 793, behind other writes 879, 797 and 816. Of fewer bytes a head the streamed scan is ahead by itself (256 of 16384 505
// and 502, keys alone of 32768 579 and 503), of more as well (of 65536 1831 and 1775, after 600 MB 1806; fp32 of 32768 1807 and 1791), and with several workgroups a head (128 of 32768 509 and 509, 64 311 and 272).
constexpr int64_t kStartBytes = 800000000, kStartHeadBytes = 10000000, kStartHeadBytesMost = 26000000;

CachedShares cached_shares(const curdkv_ctx* ctx, int64_t n, int64_t kept, bool one_workgroup) {
    const int64_t bytes = scan_bytes(ctx, n), head = bytes / ctx->heads;
    const auto part = [&](int64_t of) { return (int)(of < bytes ? of * 256 / bytes : 256); };
    return {one_workgroup && head >= kStartHeadBytes && head <= kStartHeadBytesMost ? part(kStartBytes) : 0, many_kept(ctx, n, kept) ? part(kStayBytes) : 0};
}

hipError_t configure_kernels(curdkv_ctx* ctx) {
    (void)ctx;                     // every scoring kernel uses static LDS only
    return hipSuccess;
}

hipError_t launch_scores(const curdkv_ctx* ctx, const void* K, const void* V, int64_t n,
                         float* scores, hipStream_t stream, bool normalise, int* blocks_per_head,
                         int64_t out_stride, int64_t out_offset, double* sums, bool restart,
                         bool* summed, bool with_hist, int32_t n_sink, int64_t kept, bool uneven) {
    if (out_stride <= 0) out_stride = n;
    const bool few = few_tokens(ctx, n, sums != nullptr) && !with_hist;
    const bool stream_past = stream_rows(ctx, n, kept, uneven);
    const int bph = few ? few_blocks_per_head(ctx, n, sums != nullptr) : pick_blocks_per_head(ctx, n, stream_past, with_hist ? split_hists(ctx) : kMaxBlocksPerHead);
    if (blocks_per_head) *blocks_per_head = bph;
    if (bph != 1) sums = nullptr;                 // several blocks per head: the caller adds the partials
    if (summed) *summed = sums != nullptr;
    const int rs = restart ? 1 : 0;
    const int hists = with_hist ? split_hists(ctx) : 0;
    if (with_hist) {
        // a workgroup's tokens (at most two stages of its waves here) must stay below 65536: 16-bit counts
        const int64_t tiles = (n + kTileTokens - 1) / kTileTokens;
        if (bph > hists || (tiles + bph - 1) / bph + 16 > 65535 / kTileTokens) return hipErrorInvalidValue;
    }
    uint32_t* hist = with_hist ? split_hist(ctx) : nullptr;
    uint32_t* coarse = with_hist ? split_coarse(ctx) : nullptr;
    const CachedShares share = cached_shares(ctx, n, kept, bph == 1);
    const dim3 grid((unsigned)(ctx->heads * bph));
    float* part = ctx->d_partial;
    auto launch = [&](auto cb, auto src, auto proj, auto count) {
        constexpr int CB = decltype(cb)::value, SRC = decltype(src)::value;
        constexpr bool PROJ = decltype(proj)::value, COUNT = decltype(count)::value;
        const int64_t steps = (n + 15) / 16;
        const bool bf16 = ctx->cfg.dtype == CURDKV_DTYPE_BF16;
        if (PROJ && !COUNT && few) {
            auto launch_few = [&](auto f32) {
                using Word = typename FewOperand<decltype(f32)::value>::Word;
                scores_few_kernel<decltype(f32)::value, CB, SRC><<<grid, (SRC == kSrcKV ? 2 : 1) * CB * 64, 0, stream>>>(
                    (const Word*)K, (const Word*)V, (const Word*)ctx->d_G, scores, part, (int32_t)n, bph,
                    (int32_t)((steps + bph - 1) / bph), out_stride, out_offset, sums, rs);
            };
            if (bf16) launch_few(std::false_type{});
            else launch_few(std::true_type{});
        } else if (bf16) {
            auto launch_bf16 = [&](auto past) {
                scores_bf16_kernel<CB, SRC, PROJ, COUNT, decltype(past)::value><<<grid, 256, 0, stream>>>(
                    (const uint4*)K, (const uint4*)V, (const uint4*)ctx->d_G, scores, part, n, bph, out_stride, out_offset, sums, rs,
                    hist, coarse, hists, n_sink, share);
            };
            if (!stream_past) launch_bf16(std::integral_constant<int, kStreamNone>{});
            else if (share.start == 0 && share.end == 0) launch_bf16(std::integral_constant<int, kStreamAll>{});
            else launch_bf16(std::integral_constant<int, kStreamParts>{});
        } else {
            auto launch_f32 = [&](auto split, auto past) {
                constexpr bool SPLIT = decltype(split)::value;
                scores_f32_kernel<CB, SRC, PROJ, COUNT, SPLIT, decltype(past)::value><<<grid, ShapeF32<CB, SPLIT>::kWaves * 64, 0, stream>>>(
                    (const float4*)K, (const float4*)V, (const float4*)ctx->d_G, scores, part, n, bph, out_stride, out_offset, sums, rs,
                    hist, coarse, hists, n_sink, share);
            };
            if constexpr (CB > 2) launch_f32(std::true_type{}, std::false_type{});
            else if constexpr (PROJ) {
                if (!f32_split(ctx, n)) launch_f32(std::false_type{}, std::false_type{});
                else if (stream_past) launch_f32(std::true_type{}, std::true_type{});
                else launch_f32(std::true_type{}, std::false_type{});
            } else launch_f32(std::false_type{}, std::false_type{});
        }
    };
    auto by_count = [&](auto cb, auto src, auto proj) {
        if (with_hist) launch(cb, src, proj, std::true_type{});
        else launch(cb, src, proj, std::false_type{});
    };
    auto by_source = [&](auto cb, auto proj) {
        switch (ctx->cfg.score_source) {
            case CURDKV_SCORE_KEY: by_count(cb, std::integral_constant<int, kSrcK>{}, proj); break;
            case CURDKV_SCORE_VALUE: by_count(cb, std::integral_constant<int, kSrcV>{}, proj); break;
            default: by_count(cb, std::integral_constant<int, kSrcKV>{}, proj); break;
        }
    };
    if (ctx->cfg.no_projection) {
        by_source(std::integral_constant<int, 2>{}, std::false_type{});
    } else {
        switch (ctx->col_blocks) {   // 16-column MFMA blocks = 2 per 32 padded columns
            case 1: by_source(std::integral_constant<int, 2>{}, std::true_type{}); break;
            case 2: by_source(std::integral_constant<int, 4>{}, std::true_type{}); break;
            default: by_source(std::integral_constant<int, 8>{}, std::true_type{}); break;
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !normalise) return e;
    int64_t nb = (n + 1023) / 1024;
    if (nb > 64) nb = 64;
    normalise_kernel<<<dim3((unsigned)(nb * ctx->heads)), 256, 0, stream>>>(scores, ctx->d_partial, n, bph, (int)nb);
    return hipGetLastError();
}

// Decode-phase bookkeeping: running sum of a head's un-normalised scores, and the
// normalisation by it.  Partial sums are added in a fixed order, in double: up to seven one after the other, a thread
// per head, so that one or two workgroups do it all; more by a wave per head.  A chain of loads against waves spread
// over the chip, us per curdkv_scores_append: 64 heads of 512 tokens (2 sums each) 8.4 against 8.7, of 2048 (4 sums)
// 15.8 and 16.2; 8 heads of 1159 (5 sums) 8.3 and 8.7, of 2048 (8 sums) 8.45 and 8.2, of 8192 (32 sums) 10.3 and 9.1; 1 head of 16384 (64 sums) 11.5 and 8.0.
constexpr int kFewPartials = 7;

__global__ __launch_bounds__(256) void accumulate_few_kernel(const float* __restrict__ partial, int blocks_per_head,
                                                             double* __restrict__ sums, int heads, int reset) {
    const int head = blockIdx.x * 256 + threadIdx.x;
    if (head >= heads) return;
    double total = 0.0;
    for (int i = 0; i < blocks_per_head; ++i) total += (double)partial[(size_t)head * kMaxBlocksPerHead + i];
    sums[head] = (reset ? 0.0 : sums[head]) + total;
}

__global__ __launch_bounds__(256) void accumulate_sums_kernel(const float* __restrict__ partial, int blocks_per_head,
                                                              double* __restrict__ sums, int heads, int reset) {
    const int head = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (head >= heads) return;
    const double total = wave_total(head_partial(partial + (size_t)head * kMaxBlocksPerHead, blocks_per_head));
    if ((threadIdx.x & 63) == 0) sums[head] = (reset ? 0.0 : sums[head]) + total;
}

__global__ __launch_bounds__(256) void normalise_sums_kernel(const float* __restrict__ raw,
                                                             const double* __restrict__ sums,
                                                             int64_t stride, int64_t n,
                                                             float* __restrict__ scores,
                                                             int chunks_per_head) {
    const int head = blockIdx.x / chunks_per_head;
    const int chunk = blockIdx.x - head * chunks_per_head;
    const double tot = sums[head];
    const float* src = raw + (size_t)head * stride;
    float* dst = scores + (size_t)head * n;
    constexpr int kInFlight = 4;                   // loads issued before the first store: all there are up to 65536 tokens
    const int64_t step = (int64_t)chunks_per_head * blockDim.x;
    for (int64_t j0 = (int64_t)chunk * blockDim.x + threadIdx.x; j0 < n; j0 += kInFlight * step) {
        float v[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int64_t j = j0 + u * step;
            v[u] = j < n ? src[j] : 0.f;
        }
        const bool zero = !(tot > 0.0);
        const float inv = zero ? 0.f : head_reciprocal(tot);
        const float uniform = (float)(1.0 / (double)n);
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int64_t j = j0 + u * step;
            if (j < n) dst[j] = zero ? uniform : v[u] * inv;
        }
    }
}

hipError_t launch_accumulate(const curdkv_ctx* ctx, int blocks_per_head, double* sums, bool reset,
                             hipStream_t stream) {
    if (blocks_per_head <= kFewPartials)
        accumulate_few_kernel<<<dim3((unsigned)((ctx->heads + 255) / 256)), 256, 0, stream>>>(
            ctx->d_partial, blocks_per_head, sums, ctx->heads, reset ? 1 : 0);
    else
        accumulate_sums_kernel<<<dim3((unsigned)((ctx->heads + 3) / 4)), 256, 0, stream>>>(
            ctx->d_partial, blocks_per_head, sums, ctx->heads, reset ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_normalise_sums(const curdkv_ctx* ctx, const float* raw, const double* sums,
                                 int64_t stride, int64_t n, float* scores, hipStream_t stream) {
    int64_t nb = (n + 1023) / 1024;
    if (nb > 64) nb = 64;
    normalise_sums_kernel<<<dim3((unsigned)(nb * ctx->heads)), 256, 0, stream>>>(raw, sums, stride, n, scores, (int)nb);
    return hipGetLastError();
}

hipError_t launch_fold(const curdkv_ctx* ctx, const float* scores_q, int64_t n, float* scores,
                       hipStream_t stream) {
    int64_t nb = (n + 1023) / 1024;
    if (nb > 64) nb = 64;
    fold_kernel<<<dim3((unsigned)(nb * ctx->heads)), 256, 0, stream>>>(scores_q, scores, n, ctx->cfg.group_size, (int)nb);
    return hipGetLastError();
}

}  // namespace curdkv
