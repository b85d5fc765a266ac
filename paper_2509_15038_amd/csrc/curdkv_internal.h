// Internal declarations shared by the host API and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "curdkv.h"

namespace curdkv {

constexpr int kHeadDim = 128;          // d the kernels are written for
constexpr int kColBlock = 32;          // sketch columns per MFMA tile (M of the 32x32 tile)
constexpr int kMaxColBlocks = 4;       // r padded to 32, 64 or 128
constexpr int kMaxBlocksPerHead = 256; // partial sums kept per (layer, group): one head can have a workgroup per compute unit
constexpr int kTileTokens = 32;        // tokens per wave tile
constexpr int kCompactRowsPerBlock = 128;  // output rows per entry of the gather's table of heads
constexpr int kFusedGatherTokens = 2048;       // curdkv_compress: heads up to which the fused kernel also gathers, whatever is kept on average,
constexpr int kFusedGatherRows = 800, kFusedGatherPercent = 9;   // longer ones: up to so many rows kept, and so much of the head more,
constexpr int kFusedGatherLongShare = 10;                        // or, where the scan's start goes through the caches (cached_shares), a tenth of it;
constexpr int kFusedUnevenRows = 512, kFusedUnevenRowsLong = 256, kFusedUnevenRowsRounds = 384;    // and a head at most so many more than the average (Rounds: more heads than units)

struct BlockInfo {                     // for gather block b, whose first output row is b*128:
    int64_t head_end;                  //   offsets[head + 1]
    int32_t head;                      //   the head that owns that row
    int32_t pad;
};

// Per-layer state of the head-wise budget allocation (adaptive_kernels.hip), in its workspace.
struct AdaLayerState {
    uint32_t bin;                      // the histogram bin that holds the layer's threshold
    uint32_t pad[3];
};

// Device copy of the offsets, refreshed when they change, followed by the
// per-gather-block table.
struct Plan {
    int64_t* d_offsets = nullptr;      // [heads + 1]
    BlockInfo* d_block_info = nullptr; // [max_blocks]
    char* d_buf = nullptr;             // holds both
    char* h_staging = nullptr;         // pinned, same layout
    size_t max_blocks = 0;
    std::vector<int64_t> cached;       // what d_offsets holds (after the queued copy)
    bool valid = false;
    hipEvent_t copied = nullptr;       // recorded after the last staging -> device copy
    bool copy_pending = false;
    hipStream_t copy_stream = nullptr; // the stream that copy was queued on
};

}  // namespace curdkv

struct curdkv_ctx {
    curdkv_config cfg;
    int device = 0;
    int heads = 0;                     // layers * kv_heads
    int col_blocks = 0;                // padded sketch_dim / 32 (1, 2 or 4)
    size_t g_elems_per_head = 0;       // packed operand elements per (layer, group)
    char* d_slab = nullptr;            // the one allocation that the following lie in (d_zero_offsets and d_scores_ws excepted)
    void* d_G = nullptr;               // packed sketches, storage type
    float* d_partial = nullptr;        // [heads, kMaxBlocksPerHead]
    int64_t* d_zero_offsets = nullptr; // [heads + 1] zeros: "keep nothing", for the scores-only use of the fused kernel
    void* d_adaptive_ws = nullptr;     // histograms, key segments and per-layer state of the head-wise budget allocation
    curdkv::BlockInfo* d_adaptive_blocks = nullptr;  // gather block table built on the device (curdkv_compress_adaptive)
    void* d_split_ws = nullptr;        // histograms and bitmaps of the split selection (split_select.hip)
    float* d_raw_ws = nullptr;         // products of few, short heads on their way to select_gather_kernel
    float* d_scores_ws = nullptr;      // [heads, max_tokens], allocated when curdkv_compress needs it
    int lds_limit = 0;                 // max dynamic LDS per workgroup, bytes
    int num_cu = 0;
    std::vector<uint8_t> sketch_outside;   // per (layer, group): a sketch of the caller's that sketch_splits refuses,
    int sketches_outside = 0;              // and how many there are
    curdkv::Plan plan;
};

namespace curdkv {

// sketch_host.cpp
void sketch_values(const curdkv_config& cfg, int layer, int head, float* G /*[d*r], rounded*/);
void round_to_storage(float* G, size_t count, int dtype);
bool sketch_splits(const float* G, size_t count);
// Pack row-major G[d][r] (already rounded) into the A-operand layout of one head.
void pack_sketch(const curdkv_config& cfg, int col_blocks, const float* G, void* packed);
size_t packed_elems(int col_blocks);

// kernel launchers; all return hipGetLastError() after the launch
// normalise = false leaves the un-normalised products in `scores` and the per-block
// sums in ctx->d_partial (*blocks_per_head of them per head) for launch_select to scale.
hipError_t launch_scores(const curdkv_ctx* ctx, const void* K, const void* V, int64_t n,
                         float* scores, hipStream_t stream, bool normalise = true,
                         int* blocks_per_head = nullptr, int64_t out_stride = 0, int64_t out_offset = 0,
                         double* sums = nullptr, bool restart = false, bool* summed = nullptr,
                         bool with_hist = false, int32_t n_sink = 0, int64_t kept = 0, bool uneven = false);
// with_hist: every workgroup also leaves its counts of the products of tokens n_sink and up for the
// split selection (split_select.hip), which must apply to n.
// kept: rows that the call reads again to gather them; uneven: by select_gather_kernel, from budgets that even_budgets refuses.
// sums (device, [heads]) given: where one block scores a whole head, the kernel itself adds the
// head's total to sums[head] (after zeroing it if `restart`) and *summed is set; otherwise the
// caller adds the partial sums (launch_accumulate).
int64_t scan_bytes(const curdkv_ctx* ctx, int64_t n);                  // that a scan of n tokens a head reads
bool many_kept(const curdkv_ctx* ctx, int64_t n, int64_t kept);        // a quarter of the rows or more
// In 256ths: how much of a streamed scan, at its start and at its end, goes through the caches all the same; kept: rows that a gather reads afterwards; one_workgroup: scans a head.
struct CachedShares { int start, end; };
CachedShares cached_shares(const curdkv_ctx* ctx, int64_t n, int64_t kept, bool one_workgroup);
hipError_t launch_accumulate(const curdkv_ctx* ctx, int blocks_per_head, double* sums, bool reset,
                             hipStream_t stream);
hipError_t launch_normalise_sums(const curdkv_ctx* ctx, const float* raw, const double* sums,
                                 int64_t stride, int64_t n, float* scores, hipStream_t stream);
hipError_t launch_fold(const curdkv_ctx* ctx, const float* scores_q, int64_t n, float* scores,
                       hipStream_t stream);
// scale_blocks > 0: `scores` holds un-normalised products; the kernel divides them by
// the head's sum (ctx->d_partial, scale_blocks partial sums per head), selects on the
// result and writes it back, which is what normalisation followed by selection gives
// (write_scaled = false: selects on the divided values but leaves `scores` as they are, for
// callers that do not want the scores).
// max_budget: the largest of the heads' budgets; negative: they exist on the device only.  total: their sum.
// known_thresholds (device, one {key, need} pair per head as the budget allocation leaves them,
// adaptive_thresholds): heads whose entry is valid skip the search for their threshold.
// gather given: the selection may copy the kept rows itself; gather->done says whether it has.
// hists > 0: so many histograms per head, of the un-normalised scores, have been made by launch_scores for the split selection.
struct SelectGather {
    const void *K, *V;
    void *K_out, *V_out;
    int64_t total;                     // rows kept, all heads
    bool done;
};
// The largest budget is at most a quarter above the average (max_budget < 0: not known).  Otherwise the workgroups that gather or list a head's rows are spread over
// all XCDs: 4 heads of 99162 tokens, half kept, Dirichlet budgets, split_emit_kernel 39.2 us so, 50.5 with two XCDs a head.
inline bool even_budgets(const curdkv_ctx* ctx, int64_t max_budget, int64_t total) { return max_budget >= 0 && max_budget * ctx->heads * 4 <= total * 5; }
hipError_t launch_select(const curdkv_ctx* ctx, float* scores, int64_t n, int32_t n_sink,
                         const int64_t* d_offsets, int64_t max_budget, int64_t total, int32_t* indices, hipStream_t stream,
                         int scale_blocks = 0, bool write_scaled = true,
                         const void* known_thresholds = nullptr, SelectGather* gather = nullptr, int hists = 0);
// Few, short heads, one call: selection and gather in one launch.  `raw`: the un-normalised products (ctx->d_raw_ws);
// scores: where the normalised ones go, or nullptr.  max_budget < 0: the budgets exist on the device only.
bool select_gather_wanted(const curdkv_ctx* ctx);      // the context needs the workspace
size_t select_gather_workspace_bytes(const curdkv_ctx* ctx);
bool select_gather_applicable(const curdkv_ctx* ctx, int64_t n, int64_t total);
hipError_t launch_select_gather(const curdkv_ctx* ctx, const float* raw, float* scores, int64_t n, int32_t n_sink,
                                const int64_t* d_offsets, int64_t max_budget, int32_t* indices, hipStream_t stream,
                                int scale_blocks, const SelectGather& gather, const void* known_thresholds = nullptr);
// split_select.hip: the same for long heads, several workgroups per head (workspace ctx->d_split_ws).
// hists > 0: step 1's histograms, so many of them per head, have been made by launch_scores; otherwise they are made here.
bool split_wanted(const curdkv_ctx* ctx);              // some n <= max_tokens may take it: the context needs the workspace
bool split_applicable(const curdkv_ctx* ctx, int64_t n, bool one_call);   // one_call: scores not normalised yet, histograms from launch_scores
size_t split_workspace_bytes(const curdkv_ctx* ctx);
int split_hists(const curdkv_ctx* ctx);                // histograms per head there is room for
uint32_t* split_hist(const curdkv_ctx* ctx);           // [heads][split_hists][2048], two counts to a word
uint32_t* split_coarse(const curdkv_ctx* ctx);         // [heads][split_hists][256]
constexpr int kSplitMaxHeads = 128;                    // (layer, group) pairs the split is used for (its workspace takes 9 KB per histogram, 64 per pair up to 32 pairs and 32 beyond, and 32 KB of bitmaps at most: 0.62 or 0.33 MB a pair)
hipError_t launch_split_select(const curdkv_ctx* ctx, float* scores, int64_t n, int32_t n_sink,
                               const int64_t* d_offsets, int64_t max_budget, int64_t total, int32_t* indices, hipStream_t stream,
                               int scale_blocks, bool write_scaled, const void* known_thresholds, SelectGather* gather, int hists);
bool split_counts_in_scan(const curdkv_ctx* ctx, int64_t n);      // one call: the histograms are launch_scores' to make
hipError_t launch_compact(const curdkv_ctx* ctx, const void* K, const void* V, int64_t n,
                          const int32_t* indices, const int64_t* d_offsets, int64_t total,
                          void* K_out, void* V_out, hipStream_t stream,
                          const BlockInfo* block_info = nullptr);   // default: the table of the host-side plan
hipError_t configure_kernels(curdkv_ctx* ctx);
hipError_t configure_fused(curdkv_ctx* ctx);
hipError_t configure_adaptive(curdkv_ctx* ctx);
size_t adaptive_workspace_bytes(const curdkv_ctx* ctx);
// workspace: adaptive_workspace_bytes(ctx) bytes of device memory; nothing in it has to be
// cleared beforehand, and its contents mean nothing after the call.
// hist_ready: the per-head histograms (adaptive_hist_buffer) and their sums per exponent (adaptive_coarse_buffer) have been
// written by a kernel launched earlier on the stream (launch_fused with hist_out); otherwise a kernel of this call makes them
// from `scores`, which it normalises first where scale_blocks > 0 (as in launch_select).
// offsets, block_info (device) given: where budgets are allotted layer-wide, the same launch
// also writes the budgets' prefix sums (every layer keeps kv_heads*k rows) and the gather's
// block table, and *planned is set; where every head gets the same budget they are left to
// launch_adaptive_plan and *planned stays false.
bool adaptive_allots(int32_t k, int32_t sp, long long R);      // otherwise every head gets the same, and `scores` is not looked at
hipError_t launch_adaptive(const curdkv_ctx* ctx, void* workspace, float* scores, int64_t n, int32_t k,
                           int32_t sp, int32_t g, long long R, int32_t* budgets, hipStream_t stream,
                           bool hist_ready = false, int scale_blocks = 0, int64_t* offsets = nullptr,
                           BlockInfo* block_info = nullptr, bool* planned = nullptr);
uint32_t* adaptive_hist_buffer(const curdkv_ctx* ctx, void* workspace);
uint32_t* adaptive_coarse_buffer(const curdkv_ctx* ctx, void* workspace);
// per head {threshold key, ties to keep} after launch_adaptive has allotted budgets layer-wide
// (key 0xFFFFFFFF where a head's budget comes from its safeguard, not from the layer's threshold)
const void* adaptive_thresholds(const curdkv_ctx* ctx, void* workspace);
// The static device array that serves as that workspace for curdkv_adaptive_budgets_noalloc:
// its address on `device` (looked up by adaptive_static_workspace_init, which curdkv_create
// calls with the device current), and the number of (layer, group) pairs it is sized for.
hipError_t adaptive_static_workspace_init(int device);
void* adaptive_static_workspace(int device);
int adaptive_static_max_heads();
// offsets[i] = budgets[0] + .. + budgets[i-1], kept within [0, total] (offsets[heads] = total), and
// the gather block table for them; everything on the device.
hipError_t launch_adaptive_plan(const curdkv_ctx* ctx, const int32_t* budgets, int64_t n, int64_t total,
                                int64_t* offsets, BlockInfo* block_info, hipStream_t stream);
bool fused_applicable(const curdkv_ctx* ctx, int64_t n);
// hist_out (device, [heads][4096]) and coarse_out ([heads][128]) given: the kernel also writes every head's histogram of the
// candidates' keys (tokens n_sink and up) over the 4096 bins of the selection (select_device.h)
// and its sums per exponent, for the head-wise budget allocation that follows it.
hipError_t launch_fused(const curdkv_ctx* ctx, const void* K, const void* V, int64_t n, int32_t n_sink,
                        const int64_t* d_offsets, float* scores, int32_t* indices, void* K_out,
                        void* V_out, hipStream_t stream, int64_t kept, uint32_t* hist_out = nullptr,
                        uint32_t* coarse_out = nullptr);
// kept: rows that the call gathers, by this kernel (indices given) or after it.

}  // namespace curdkv
