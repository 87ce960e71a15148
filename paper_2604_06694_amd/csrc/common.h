// Shared declarations of the gfx950 kernels behind the AudioKV C ABI.
// Device code only needs hip_runtime; nothing here depends on torch.
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

#include "audiokv.h"

namespace audiokv {

// Geometry handed to kernels by value.
struct Geom {
    int n_items;
    int H_q;
    int H_kv;
    int G;          // H_q / H_kv
    int D;          // head_dim
    int W;          // window
    int pool_kernel;
    int pool_mode;
    int causal;
    int layout;     // AUDIOKV_LAYOUT_*
    float c_log2;   // softmax scale * log2(e): logits are handled in base-2 units
    int cutoff_mode;   // AUDIOKV_CUTOFF_*
    int taper_bins;    // cosine roll-off bins after k*
    // explicit K/V strides in elements (all zero: the packed layout named by `layout`)
    int64_t s_item, s_head, s_tok;
};

// Elements between consecutive tokens of one head.
__device__ __forceinline__ int64_t kv_tok_stride(const Geom& g) {
    if (g.s_tok) return g.s_tok;
    return g.layout == AUDIOKV_LAYOUT_HEAD_MAJOR ? (int64_t)g.D : (int64_t)g.H_kv * g.D;
}

// Where head (item, h), token j starts inside the K/V buffers (in elements). item_tok0 = cu_seqlens[item].
__device__ __forceinline__ int64_t kv_row_offset(const Geom& g, int item, int64_t item_tok0, int L, int h, int j) {
    if (g.s_tok) return (int64_t)item * g.s_item + (int64_t)h * g.s_head + (int64_t)j * g.s_tok;
    const int64_t base = item_tok0 * g.H_kv * g.D;
    if (g.layout == AUDIOKV_LAYOUT_HEAD_MAJOR)
        return base + ((int64_t)h * L + j) * g.D;
    return base + ((int64_t)j * g.H_kv + h) * g.D;
}

// Inclusive sum over the lanes of a full wave, in six data-parallel-primitive steps (no LDS).
__device__ __forceinline__ int wave_incl(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr 1, 2, 4, 8: prefixes within 16 lanes
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast 15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast 31 into rows 2 and 3
    return x;
}

// Workgroups of `threads` threads for each of n parts of a launch: as many as wanted, but a launch holds fewer than 2^32 threads,
// and parts of it go along with others: half of that at most. The kernels that ask stride over what is left.
inline int blocks_per_part(long long wanted, long long n, int threads = 256) {
    const long long most = n > 0 ? (1LL << 31) / threads / n : wanted;
    return (int)(wanted < 1 || most < 1 ? 1 : wanted < most ? wanted : most);
}

// ---- launchers (defined in the .hip files, called from api.hip) ------------

constexpr int kAllocateWaveHeads = 128;    // pools up to this size are allocated by one wave
// Arguments of launch_allocate, for callers that let the allocation ride along with another launch.
struct AllocateJob {
    const float* weights; int n_segments, heads_per_segment, weight_group; const int32_t* cu_seqlens;
    double ratio, floor_frac; int32_t* budgets; int32_t* cu_budgets;
};
struct ConvFilterJob;      // taps of the smoothing's filter (conv_filter.h)

// How a sweep of score cuts the heads into key ranges, one workgroup each: as many for every head, or, for few items of different
// lengths, ranges of as many keys each, range c of item i, head h being part (number of ranges of the items before + c) * H_kv + h.
struct ScoreRanges {
    int per_head = 1;        // as many for every head: how many
    int keys = 0;            // ranges of one size: keys of each, whole tiles (0: as many for every head)
    double per_key = 0.;     // 1 / keys
    long long parts = 1;     // workgroups of the sweep, and sets of row statistics of sweep 1
    // ranges of a head: the quotient rounded up, in float64 and off the whole numbers, so that it is exact (host and device agree,
    // and with integer divisions planning for 48 lengths took 25 us)
    __host__ __device__ int of_length(int L) const { return (int)(((double)L + (double)keys - 0.5) * per_key); }
};
constexpr int kCountedItems = 64;        // items that ranges of one size can have: a lane each
// The ranges of sweep 1; a pure function of the batch so that the workspace query and the launch agree.
// max_parts: not more parts than these, if one range for every head is not more already.
ScoreRanges score_ranges(int H_kv, int n_items, const int32_t* seqlens_host, int rows, int D, long long max_parts = LLONG_MAX);
// Padded row count (multiple of the MFMA row tiling) for G*W window rows; 0 if unsupported.
int score_padded_rows(int rows, int D);

// ranges: score_ranges() of the batch.
// between_sweeps: optional event recorded on `s` after the first sweep (timing aid), or nullptr.
// lse: optional fp32 [items][H_q][W] natural-log softmax denominators of the window rows; given, sweep 1 is skipped.
// ride_along, ride_taps: optional allocation (pools of at most kAllocateWaveHeads heads) and filter taps to run in extra
// workgroups of the first sweep.
hipError_t launch_score(const Geom& g, const void* q_win, const void* k, const int32_t* cu_seqlens,
                        const int32_t* seqlens_host, const ScoreRanges& ranges, float* stats_ws, float* raw_out, hipStream_t s,
                        hipEvent_t between_sweeps = nullptr, const float* lse = nullptr,
                        float* raw_second = nullptr, size_t raw_elems = 0, const AllocateJob* ride_along = nullptr,
                        const ConvFilterJob* ride_taps = nullptr);
// More than 448 window rows (d <= 128): sweep 2 runs as two launches and needs a second buffer of the size of the
// scores (raw_second, raw_elems floats).
bool score_needs_second_raw(int rows, int D);
// raw: inside a workspace that extends 16 floats to either side of every head
hipError_t launch_pool(const Geom& g, const float* raw, const int32_t* cu_seqlens, int max_L,
                       float* pooled, hipStream_t s);

hipError_t launch_allocate(const Geom& g, const float* weights, int n_segments, int heads_per_segment,
                           int weight_group, const int32_t* cu_seqlens, double ratio, double floor_frac,
                           int32_t* budgets, int32_t* cu_budgets, hipStream_t s);

// pool_on_load: input holds un-pooled scores and the pooling of Geom is applied while loading.
bool smooth_supported(int L);
// Global-memory scratch of the smoothing: what the transforms of lengths that are not powers of two need
// (_required: 0 when every length is a power of two), plus, for calls with few heads, room to spread a
// power-of-two head over several workgroups (_bytes: the sum; what the workspace query reserves).
size_t smooth_workspace_bytes(const int32_t* seqlens_host, int n_items, int H_kv);
size_t smooth_workspace_required(const int32_t* seqlens_host, int n_items, int H_kv);
// kstar_out (may be null): the cutoff bin of every head; cutoffs_only stops after writing it. workspace_bytes: what
// `workspace` holds (at least _required; with less than _bytes every power-of-two head runs in one workgroup).
// join (conv.h): if given, the last step of some heads may be left to launch_select, and `out` without their result.
// select (select_head.h): if given, the launch may select as well, and says so.
struct ConvJoin;
struct SelectJob;
hipError_t launch_smooth(const Geom& g, const float* in, bool pool_on_load, const int32_t* cu_seqlens,
                         const int32_t* seqlens_host, int n_items, double cutoff_frac, double alpha,
                         float* out, void* workspace, size_t workspace_bytes, int32_t* kstar_out, bool cutoffs_only,
                         hipStream_t s, bool filters_ready = false, ConvJoin* join = nullptr, SelectJob* select = nullptr);
// What lengths that are not powers of two need that depends on the lengths and the cutoff only: launch_smooth_filters
// prepares it in the workspace (launch_smooth does it itself unless told that it is ready). smooth_filters says how much
// that is: several launches (long_work, worth a stream of its own), or the taps alone, which can ride along elsewhere,
// or nothing.
struct SmoothFilters;
SmoothFilters smooth_filters(const Geom& g, const int32_t* cu_seqlens, const int32_t* seqlens_host, int n_items,
                             double cutoff_frac, void* workspace);
hipError_t launch_smooth_filters(const Geom& g, const int32_t* cu_seqlens, const int32_t* seqlens_host, int n_items,
                                 double cutoff_frac, void* workspace, hipStream_t s);

// single-query attention over the packed cache
bool decode_supported(int G);
size_t decode_workspace_bytes(const Geom& g, long long total_rows);
hipError_t launch_decode(const Geom& g, const void* q, const void* k_cache, const void* v_cache,
                         const int32_t* cu_budgets, long long total_rows, float* out, void* workspace, hipStream_t s);

bool select_supported(int L);
// whether launch_select can combine what smoothing left
bool select_joins(int max_L);
hipError_t launch_select(const Geom& g, const float* scores, const int32_t* budgets, const int32_t* cu_budgets,
                         const int32_t* cu_seqlens, int max_L, int32_t* indices, hipStream_t s, const ConvJoin* join = nullptr);

// total_tokens: of all items, total_rows: kept, of all heads
hipError_t launch_compact(const Geom& g, const void* k, const void* v, const int32_t* indices,
                          const int32_t* cu_budgets, const int32_t* cu_seqlens, int64_t total_tokens, int64_t total_rows,
                          void* k_out, void* v_out, hipStream_t s);

}  // namespace audiokv
