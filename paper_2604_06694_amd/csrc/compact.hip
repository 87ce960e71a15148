// Stage 5: gather the retained K/V rows into the packed cache.
// Pure data movement: every row is d*2 bytes (128-512 B), moved as 16-byte
// vectors so that a row is read and written by 8-32 adjacent lanes.
//
// Bound by HBM, and for small caches by the chain head -> index -> row -> store.
// A thread moves one vector of K and one of V and the waves do the rest: with
// so few registers a CU holds 32 of them. (Eight rows per thread, the loads of
// all in flight, is slower at every size: 3.3 k rows 6.3 us against 3.7, 22 k 9.7
// against 6.2, 52 k 15.0 against 11.7, 1.47 M 266 against 246, 6.1 TB/s.)
#include "common.h"

namespace audiokv {

namespace {

constexpr int kThreads = 256;

// Largest g with cu_b[g] <= p (cu_b is a non-decreasing exclusive scan, cu_b[n] = total > p; p uniform). Every round
// probes 64 heads at equal distances, one per lane: one load latency for up to 64 heads, two up to 4096.
__device__ __forceinline__ int head_of_row(const int32_t* __restrict__ cu_b, int n_heads, int p) {
    int head = 0;
    for (int span = n_heads; span > 1;) {
        const int step = (span + 63) >> 6;
        const int probe = head + (int)(threadIdx.x & 63) * step;
        const bool at_or_before = probe < head + span && cu_b[min(probe, n_heads - 1)] <= p;
        const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(at_or_before));   // a prefix of the lanes
        const int skip = n > 0 ? (n - 1) * step : 0;
        head += skip;
        span = min(step, span - skip);
    }
    return __builtin_amdgcn_readfirstlane(head);
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // 16 bytes; the nontemporal builtins need a native vector

// VEC_PER_ROW: 16-byte vectors per row = D * 2 / 16. STREAM: what is read and written is too much for the memory-side cache.
// Rows of a small cache stay there for the decoding step that follows, and K may still be there from the scoring. With nontemporal
// accesses and without (K, V and kept rows together): the gather of 8 ragged items (110 MB) 12.6 and 11.4 us, evict on one layer of
// 32768 (47 MB) 96.4 and 94.4; with a decoding step 4 layers of 8192 (94 MB) 80.4 and 77.1, 8 of 5000 (115 MB) 113 and 109;
// 8 ragged items at d = 256 (178 MB, other inputs each time) 128.1 and 131.9, 28 layers of 8192 274 and 278.
template <int VEC_PER_ROW, bool STREAM>
__global__ __launch_bounds__(kThreads) void compact_kernel(
    Geom g, const u32x4* __restrict__ k, const u32x4* __restrict__ v,
    const int32_t* __restrict__ indices, const int32_t* __restrict__ cu_b,
    const int32_t* __restrict__ cu_seq, int n_heads, int64_t first_row, int64_t total_rows,
    u32x4* __restrict__ k_out, u32x4* __restrict__ v_out)
{
    constexpr int ROWS = kThreads / VEC_PER_ROW;   // consecutive output rows of a workgroup
    const int vec = threadIdx.x % VEC_PER_ROW;     // 16-byte piece of the row
    const int64_t row0 = first_row + (int64_t)blockIdx.x * ROWS;
    // the head of the workgroup's first row is found once; a later row walks forward from there
    int gh = head_of_row(cu_b, n_heads, (int)row0);
    // (a row past the end is the last row again, which is not stored: no branch around the loads)
    const int64_t p = row0 + threadIdx.x / VEC_PER_ROW, pc = min(p, total_rows - 1);
    const int idx = indices[pc];
    while (gh + 1 < n_heads && cu_b[gh + 1] <= pc) ++gh;
    const int item = gh / g.H_kv, h = gh - item * g.H_kv;
    const int tok0 = cu_seq[item];
    const int L = cu_seq[item + 1] - tok0;
    // an index outside the item is a caller error; clamp so that it can never fault
    const int64_t src = kv_row_offset(g, item, tok0, L, h, min(max(idx, 0), L - 1)) / 8 + vec;   // strides are multiples of 8
    const u32x4 kk = STREAM ? __builtin_nontemporal_load(k + src) : k[src];
    const u32x4 vv = STREAM ? __builtin_nontemporal_load(v + src) : v[src];
    if (p < total_rows) {
        if constexpr (STREAM) {
            __builtin_nontemporal_store(kk, k_out + p * VEC_PER_ROW + vec);
            __builtin_nontemporal_store(vv, v_out + p * VEC_PER_ROW + vec);
        } else {
            k_out[p * VEC_PER_ROW + vec] = kk;
            v_out[p * VEC_PER_ROW + vec] = vv;
        }
    }
}

}  // namespace

hipError_t launch_compact(const Geom& g, const void* k, const void* v, const int32_t* indices,
                          const int32_t* cu_budgets, const int32_t* cu_seqlens, int64_t total_tokens, int64_t total_rows,
                          void* k_out, void* v_out, hipStream_t s)
{
    if (total_rows <= 0) return hipSuccess;
    const int64_t all = (total_tokens * g.H_kv + total_rows) * g.D * 4;      // bytes of K and V, whole and kept
    const bool stream = all > (128LL << 20);
    const int n_heads = g.n_items * g.H_kv;
    const int vec_per_row = g.D / 8;
    const int rows_per_block = kThreads / vec_per_row;
    // a launch holds fewer than 2^32 threads: rows beyond that (60 GB and more) take further ones
    const int64_t slab = (int64_t)rows_per_block << 23;
#define AUDIOKV_LAUNCH_COMPACT(V, S)                                                                \
    hipLaunchKernelGGL((compact_kernel<V, S>), dim3(blocks), dim3(kThreads), 0, s, g,               \
                       (const u32x4*)k, (const u32x4*)v, indices, cu_budgets, cu_seqlens, n_heads, \
                       first, total_rows, (u32x4*)k_out, (u32x4*)v_out)
    for (int64_t first = 0; first < total_rows; first += slab) {
        const int64_t rows = total_rows - first < slab ? total_rows - first : slab;
        const unsigned blocks = (unsigned)((rows + rows_per_block - 1) / rows_per_block);
        switch (vec_per_row) {
            case 8:  if (stream) AUDIOKV_LAUNCH_COMPACT(8, true); else AUDIOKV_LAUNCH_COMPACT(8, false);  break;
            case 16: if (stream) AUDIOKV_LAUNCH_COMPACT(16, true); else AUDIOKV_LAUNCH_COMPACT(16, false); break;
            case 32: if (stream) AUDIOKV_LAUNCH_COMPACT(32, true); else AUDIOKV_LAUNCH_COMPACT(32, false); break;
            default: return hipErrorInvalidValue;
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
#undef AUDIOKV_LAUNCH_COMPACT
    return hipSuccess;
}

}  // namespace audiokv
