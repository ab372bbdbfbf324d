// Visual-textual collaborative pruning and merging (Sec. 3.2.3, Eq. 5-6; Alg. 3 of arXiv
// 2601.17818): inside every cluster of visual tokens the q_c tokens with the smallest K-vector
// norm survive as "elites", the rest of the cluster is averaged into one merged token.
//
//   1. collab_rank_kernel   per token: size of its cluster and its rank inside it by
//                           (K-norm, index) ascending -> elite iff rank < q_c, with
//                           q_c = floor(|C_c| (B - N_c) / n)                       (Eq. 5)
//   2. collab_plan_kernel   per image: output row of every token (elites in ascending
//                           token index, then one merged row per cluster that has
//                           non-elites, in cluster order), row count, representative
//                           token of each row
//   3. collab_emit_kernel   per output row: copy of the elite, or the mean of the
//                           absorbed tokens (fp32 sums in ascending token order)   (Eq. 6)
//
// Everything is integer work on the given labels and fp32 norms except the means, so the
// result is deterministic; ties in the norm go to the lower index.
#include <atomic>
#include "vitcop_internal.h"
#include "device_utils.h"

namespace vitcop {

constexpr int CB_ROW_THREADS = 256;      // 4 wavefronts, one token each
constexpr int CB_PLAN_THREADS = 1024;

// B - N_c, not below 0
__device__ __forceinline__ int elite_budget(int budget, int n_clusters) { return max(0, budget - n_clusters); }

__global__ __launch_bounds__(CB_ROW_THREADS) void collab_rank_kernel(
    const int32_t* __restrict__ labels, const float* __restrict__ norms,
    const int32_t* __restrict__ n_clusters, int n, int budget, int32_t* __restrict__ elite) {
    const int b = blockIdx.y, lane = threadIdx.x & 63;
    const int i = blockIdx.x * (CB_ROW_THREADS / 64) + (threadIdx.x >> 6);
    if (i >= n) return;
    labels += (int64_t)b * n;
    norms += (int64_t)b * n;
    const int li = labels[i];
    const float ni = norms[i];
    int size = 0, rank = 0;
    for (int j = lane; j < n; j += 64) {
        const bool same = labels[j] == li;
        const float nj = norms[j];
        size += same ? 1 : 0;
        rank += (same && (nj < ni || (nj == ni && j < i))) ? 1 : 0;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        size += __shfl_xor(size, o, 64);
        rank += __shfl_xor(rank, o, 64);
    }
    if (lane == 0) {
        const int quota = (int)(((int64_t)size * elite_budget(budget, n_clusters[b])) / n);
        elite[(int64_t)b * n + i] = rank < quota ? 1 : 0;
    }
}

// One workgroup per image.  LDS: has_rest[R] / merged_row[R] and first_rest[R], R <= n.
__global__ __launch_bounds__(CB_PLAN_THREADS) void collab_plan_kernel(
    const int32_t* __restrict__ labels, int32_t* __restrict__ elite,
    const int32_t* __restrict__ n_clusters, int n, int32_t* __restrict__ assign,
    int32_t* __restrict__ out_index, int32_t* __restrict__ n_out) {
    extern __shared__ __attribute__((aligned(16))) int cb_lds[];
    __shared__ int wave_tot[CB_PLAN_THREADS / 64];
    const int tid = threadIdx.x, b = blockIdx.x;
    labels += (int64_t)b * n;
    elite += (int64_t)b * n;
    assign += (int64_t)b * n;
    out_index += (int64_t)b * n;
    const int R = min(max(n_clusters[b], 0), n);          // labels are the caller's contract; stay inside LDS anyway
    auto label_of = [&](int i) { return min(max(labels[i], 0), max(R - 1, 0)); };
    int* merged_row = cb_lds;            // first: 1 if the cluster has non-elites; then: its output row
    int* first_rest = cb_lds + n;        // lowest token index among the cluster's non-elites
    for (int c = tid; c < R; c += CB_PLAN_THREADS) {
        merged_row[c] = 0;
        first_rest[c] = 0x7fffffff;
    }
    __syncthreads();
    for (int i = tid; i < n; i += CB_PLAN_THREADS)
        if (!elite[i]) {
            merged_row[label_of(i)] = 1;                    // same value from every writer
            atomicMin(&first_rest[label_of(i)], i);
        }
    __syncthreads();

    // elites keep their order: row = number of elites before the token
    const int n_elite = block_exclusive_scan<CB_PLAN_THREADS>(
        0, n, wave_tot, [&](int i) { return elite[i]; },
        [&](int i, int f, int pos) {
            if (f) {
                assign[i] = pos;
                out_index[pos] = i;
            }
        });
    // merged rows follow, one per cluster with non-elites, in cluster order
    const int n_merged = block_exclusive_scan<CB_PLAN_THREADS>(
        0, R, wave_tot, [&](int c) { return merged_row[c]; },
        [&](int c, int f, int pos) {
            if (f) out_index[n_elite + pos] = first_rest[c];
            merged_row[c] = n_elite + pos;
        });
    __syncthreads();
    for (int i = tid; i < n; i += CB_PLAN_THREADS)
        if (!elite[i]) assign[i] = merged_row[label_of(i)];
    if (tid == 0) n_out[b] = n_elite + n_merged;
    __syncthreads();                     // the flags have been read: their first entry now says how many elites there are
    if (tid == 0 && n > 0) elite[0] = n_elite;
}

// One workgroup per (output row, image); a thread owns 8 channels.  Rows [0, n_elite) are elites, the merged ones follow.
// A chain of round trips to memory: what the row is, and which tokens go to it, are read together, then eight members'
// rows at a time (8 x 288 tokens x 4096, 36 MB: 8.7 us with the elite flag and the assignment read one after the other and
// four members at a time by half the threads, 7.6 now).
constexpr int CB_TOKENS = 1024;          // tokens looked at between two barriers

template <int THREADS>
__global__ __launch_bounds__(THREADS) void collab_emit_kernel(
    const uint16_t* __restrict__ feats, int64_t row_stride, int64_t batch_stride,
    const int32_t* __restrict__ elite, const int32_t* __restrict__ assign,
    const int32_t* __restrict__ out_index, const int32_t* __restrict__ n_out, int n, int D,
    uint16_t* __restrict__ out_feats) {
    constexpr int WAVES = THREADS / 64, CHUNKS = CB_TOKENS / THREADS;
    // merged rows, the last ones, take longest: they start first (8 x 288 tokens x 4096 9.6 -> 9.1 us, 1856 x 3584 14.5 -> 12.5)
    const int r = n - 1 - blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    feats += b * batch_stride;
    assign += (int64_t)b * n;
    uint16_t* dst = out_feats + ((int64_t)b * n + r) * D;
    const int rows = n_out[b], elites = elite[(int64_t)b * n];       // (left there by collab_plan_kernel)
    const int first = out_index[(int64_t)b * n + r];      // (of a row past the end: unused)
    int to[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) to[c] = assign[min(c * THREADS + tid, n - 1)];
    if (r >= rows) return;
    if (r < elites) {                                     // an elite row: plain copy
        const uint16_t* src = feats + (int64_t)first * row_stride;
        for (int c = tid * 8; c < D; c += THREADS * 8)
            *reinterpret_cast<uint4*>(dst + c) = *reinterpret_cast<const uint4*>(src + c);
        return;
    }
    // a merged row: list the absorbed tokens in ascending order, then average them channel by channel
    __shared__ int members[VITCOP_VIC_MAX_TOKENS];
    __shared__ unsigned found[2][CHUNKS * WAVES];         // (two: one may be read while the next is written)
    static_assert(CHUNKS * WAVES <= 64, "a count a lane");
    int count = 0;
    for (int i0 = 0; i0 < n; i0 += CB_TOKENS) {
        unsigned* counts = found[i0 / CB_TOKENS & 1];
        if (i0 > 0)
#pragma unroll
            for (int c = 0; c < CHUNKS; ++c) to[c] = assign[min(i0 + c * THREADS + tid, n - 1)];
        unsigned long long mask[CHUNKS];
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            mask[c] = __builtin_amdgcn_ballot_w64(i0 + c * THREADS + tid < n && to[c] == r);
            if (lane == 0) counts[c * WAVES + wv] = (unsigned)__builtin_popcountll(mask[c]);
        }
        __syncthreads();
        const unsigned mine = lane < CHUNKS * WAVES ? counts[lane] : 0u;
        const unsigned incl = wave_scan(mine, 0u, [](unsigned x, unsigned y) { return x + y; }), before = incl - mine;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c)
            if (mask[c] >> lane & 1u)
                members[count + __builtin_amdgcn_readlane(before, c * WAVES + wv) +
                        __builtin_amdgcn_mbcnt_hi((unsigned)(mask[c] >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask[c], 0u))] =
                    i0 + c * THREADS + tid;
        count += (int)__builtin_amdgcn_readlane(incl, 63);
    }
    __syncthreads();
    const float inv = 1.0f / (float)count;
    for (int c = tid * 8; c < D; c += THREADS * 8) {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int m0 = 0; m0 < count; m0 += 8) {               // eight members' rows in flight
            u32x4 row[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (m0 + e < count)
                    row[e] = *reinterpret_cast<const u32x4*>(feats + (int64_t)members[m0 + e] * row_stride + c);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (m0 + e < count) {
                    acc[0] += bf16_lo(row[e].x); acc[1] += bf16_hi(row[e].x);
                    acc[2] += bf16_lo(row[e].y); acc[3] += bf16_hi(row[e].y);
                    acc[4] += bf16_lo(row[e].z); acc[5] += bf16_hi(row[e].z);
                    acc[6] += bf16_lo(row[e].w); acc[7] += bf16_hi(row[e].w);
                }
        }
        uint4 o;
        o.x = pack_bf16(acc[0] * inv, acc[1] * inv);
        o.y = pack_bf16(acc[2] * inv, acc[3] * inv);
        o.z = pack_bf16(acc[4] * inv, acc[5] * inv);
        o.w = pack_bf16(acc[6] * inv, acc[7] * inv);
        *reinterpret_cast<uint4*>(dst + c) = o;
    }
}

size_t collab_workspace_bytes(int B, int n) { return 2 * up256((size_t)B * n * 4); }   // elite flags, row of every token

int launch_collab(const uint16_t* feats, int64_t row_stride, int64_t batch_stride, const int32_t* labels,
                  const int32_t* n_clusters, const float* norms, int B, int n, int D, int budget,
                  uint16_t* out_feats, int32_t* out_index, int32_t* n_out, int32_t* assign, void* ws,
                  hipStream_t s) {
    if (B == 0) return VITCOP_OK;
    int32_t* elite = static_cast<int32_t*>(ws);
    if (!assign) assign = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + up256((size_t)B * n * 4));
    if (n > 0) {
        dim3 grid((unsigned)((n + CB_ROW_THREADS / 64 - 1) / (CB_ROW_THREADS / 64)), B);
        hipLaunchKernelGGL(collab_rank_kernel, grid, dim3(CB_ROW_THREADS), 0, s, labels, norms, n_clusters, n, budget,
                           elite);
        int rc = launch_status("collab_rank");
        if (rc) return rc;
    }
    static std::atomic<bool> attr_set{false};   // set once; a second thread repeating the call is harmless
    if (!attr_set.load(std::memory_order_acquire)) {
        int rc = hip_status(hipFuncSetAttribute((const void*)collab_plan_kernel,
                                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                                2 * VITCOP_VIC_MAX_TOKENS * 4 + 16),
                            "hipFuncSetAttribute(collab_plan)");
        if (rc) return rc;
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(collab_plan_kernel, dim3(B), dim3(CB_PLAN_THREADS), (size_t)2 * n * 4 + 16, s, labels, elite,
                       n_clusters, n, assign, out_index, n_out);
    int rc = launch_status("collab_plan");
    if (rc || n == 0) return rc;
    if (D > 2048)                        // (one pass over the channels up to 4096)
        hipLaunchKernelGGL(collab_emit_kernel<512>, dim3(n, B), dim3(512), 0, s, feats, row_stride, batch_stride, elite,
                           assign, out_index, n_out, n, D, out_feats);
    else
        hipLaunchKernelGGL(collab_emit_kernel<256>, dim3(n, B), dim3(256), 0, s, feats, row_stride, batch_stride, elite,
                           assign, out_index, n_out, n, D, out_feats);
    return launch_status("collab_emit");
}

}  // namespace vitcop
