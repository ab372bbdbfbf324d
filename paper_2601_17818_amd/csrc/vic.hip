// Visual Information Clustering (Sec. 3.2.1, Eq. 2-3; Alg. 2 of arXiv 2601.17818): a
// density-peak clustering of the visual tokens that survived Stage I, constrained to
// spatial neighbours.
//
//   1. inner products of the features and their squared norms   gemm_kernel<.., GM_EPI_GRAM>
//   2. D_feat[i,j] = ||f_i - f_j||_2 from them, and
//      rho_i = sum_{j != i} exp(-(D_feat[i,j]/d_c)^2)  (Eq. 2)  vic_density_kernel
//   3. delta_i, N_i = min / argmin of D_feat[i,j] over j with rho_j > rho_i and
//      D_spatial[i,j] <= tau (Eq. 3), gamma_i = rho_i delta_i   vic_parent_kernel
//   4. the n_centers largest gamma are centres; every other token follows its
//      parent pointers N_i up to a root (a centre, or a token without parent);
//      clusters are numbered by the index of their root          vic_label_kernel
//
// Every decision (rho_j > rho_i, the minimum, the TopK of gamma) is taken on the fp32
// values this code writes out, ties going to the lower index, so the result is
// a deterministic function of those arrays.  The order of Step 4 of Alg. 2
// (tokens in decreasing density take their parent's label) is replaced by
// pointer jumping, which reaches the same labels: a parent is strictly denser
// than its child, so the parent chains have no cycles.
#include <atomic>
#include "vitcop_internal.h"
#include "device_utils.h"
#include "select_device.h"

namespace vitcop {

constexpr int VIC_ROWS = 8, VIC_THREADS = 64 * VIC_ROWS;       // a workgroup: 8 rows, one per wavefront
constexpr int VIC_COLS = 512, VIC_CPL = VIC_COLS / 64, VIC_FETCH = VIC_COLS * VIC_ROWS / 4 / VIC_THREADS;

// Workgroup -> (image, first row): every XCD (consecutive workgroup ids go to different ones) takes a contiguous range,
// so that the row blocks that share the columns' 128-byte lines meet in one L2.
__device__ __forceinline__ int vic_rows_of(int blocks, int& image) {
    const int all = gridDim.x, xcd = blockIdx.x % 8;
    const int lin = xcd * (all / 8) + min(xcd, all % 8) + blockIdx.x / 8;
    image = lin / blocks;
    return (lin - image * blocks) * VIC_ROWS;
}

// Squared distances of this workgroup's rows to 512 columns at a time, from the two halves of their inner products,
// which lie mirrored at the diagonal (launch_gram): the rows' own half is read along the rows, the other, a few
// rows of each column, goes through LDS.  f(j, d2, column(j)) is called by the lane that owns column j of its
// wavefront's row i: lane l owns columns l, l + 64, ... in order.  Latency-bound at a few hundred tokens: a round's
// loads, column(j)'s too, are in flight together.
template <typename C, typename F>
__device__ __forceinline__ void vic_distances(const float* __restrict__ gram, int64_t stride,
                                              const float* __restrict__ sq, int64_t sq_half, int n, int i0, C column, F f) {
    __shared__ float mirrored[VIC_ROWS][VIC_COLS + 4];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i = i0 + wv, ic = min(i, n - 1);               // (clamped: values that no live row or column uses)
    const float sq_i = sq[ic] + sq[sq_half + ic];
    for (int j0 = 0; j0 < n; j0 += VIC_COLS) {
        float own[VIC_CPL], sq_a[VIC_CPL], sq_b[VIC_CPL];
        decltype(column(0)) data[VIC_CPL];
        float4 col[VIC_FETCH];
#pragma unroll
        for (int q = 0; q < VIC_FETCH; ++q) {
            const int id = tid + VIC_THREADS * q, cj = id % VIC_COLS, cr = id / VIC_COLS * 4;
            col[q] = *reinterpret_cast<const float4*>(gram + (int64_t)min(j0 + cj, n - 1) * stride +
                                                      min((int64_t)i0 + cr, stride - 4));
        }
#pragma unroll
        for (int c = 0; c < VIC_CPL; ++c) {
            if (j0 + 64 * c >= n) break;                     // (uniform)
            const int j = min(j0 + 64 * c + lane, n - 1);
            sq_a[c] = sq[j];
            sq_b[c] = sq[sq_half + j];
            data[c] = column(j);
            own[c] = gram[(int64_t)ic * stride + j];
        }
        __syncthreads();                                     // the columns before have been read
#pragma unroll
        for (int q = 0; q < VIC_FETCH; ++q) {
            const int id = tid + VIC_THREADS * q, cj = id % VIC_COLS, cr = id / VIC_COLS * 4;
            mirrored[cr][cj] = col[q].x;
            mirrored[cr + 1][cj] = col[q].y;
            mirrored[cr + 2][cj] = col[q].z;
            mirrored[cr + 3][cj] = col[q].w;
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < VIC_CPL; ++c) {
            if (j0 + 64 * c >= n) break;
            const int j = j0 + 64 * c + lane;
            const float d2 = fmaxf(0.f, fmaf(-2.f, own[c] + mirrored[wv][64 * c + lane], sq_i + (sq_a[c] + sq_b[c])));
            if (i < n && j < n) f(j, i == j ? 0.f : d2, data[c]);
        }
    }
}

// Eq. 2.  A lane adds its columns in order, then the 64 lane sums of a row are combined by the fixed xor tree: the
// result does not depend on scheduling.  dist (nullable) receives the distances.
__global__ __launch_bounds__(VIC_THREADS) void vic_density_kernel(const float* __restrict__ gram, int64_t stride,
                                                                  int64_t batch, const float* __restrict__ sq,
                                                                  int64_t sq_batch, int64_t sq_half, int n,
                                                                  float neg_inv_dc2_log2e,
                                                                  float* __restrict__ rho, float* __restrict__ dist) {
    int img;
    const int i0 = vic_rows_of((n + VIC_ROWS - 1) / VIC_ROWS, img), i = i0 + (threadIdx.x >> 6);
    if (dist) dist += img * batch + (int64_t)i * stride;
    float acc = 0.f;
    vic_distances(gram + img * batch, stride, sq + img * sq_batch, sq_half, n, i0, [](int) { return 0; },
                  [&](int j, float d2, int) {
                      if (dist) dist[j] = __builtin_sqrtf(d2);
                      const float e = __builtin_amdgcn_exp2f(d2 * neg_inv_dc2_log2e);
                      acc += (j != i) ? e : 0.f;
                  });
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0 && i < n) rho[(int64_t)img * n + i] = acc;
}

// Eq. 3.  Candidates are ordered by (distance, index).
__global__ __launch_bounds__(VIC_THREADS) void vic_parent_kernel(
    const float* __restrict__ gram, int64_t stride, int64_t batch, const float* __restrict__ sq, int64_t sq_batch,
    int64_t sq_half, const float* __restrict__ pos, const float* __restrict__ rho, int n, float tau2,
    float* __restrict__ delta, int32_t* __restrict__ parent) {
    int img;
    const int i0 = vic_rows_of((n + VIC_ROWS - 1) / VIC_ROWS, img), i = i0 + (threadIdx.x >> 6), ic = min(i, n - 1);
    pos += 2 * (int64_t)img * n;
    rho += (int64_t)img * n;
    const float rho_i = rho[ic], px = pos[2 * ic], py = pos[2 * ic + 1];
    float best = INFINITY, best2 = INFINITY;                 // (best2 squared: a root only where it may matter)
    int best_j = 0x7fffffff;
    vic_distances(gram + img * batch, stride, sq + img * sq_batch, sq_half, n, i0,
                  [&](int j) { return make_float3(pos[2 * j], pos[2 * j + 1], rho[j]); },      // (pos: aligned to 4 bytes)
                  [&](int j, float d2, const float3& col) {
                      const float dx = col.x - px, dy = col.y - py;
                      if (col.z > rho_i && dx * dx + dy * dy <= tau2 && d2 < best2) {
                          const float d = __builtin_sqrtf(d2);
                          best2 = d2;
                          if (d < best) {  // j ascends within a lane: strict "<" keeps the lower index
                              best = d;
                              best_j = j;
                          }
                      }
                  });
    // the least distance of the row, then the least index that has it
    const float least = wave_reduce(best, INFINITY, [](float a, float b) { return b < a ? b : a; });
    best_j = wave_reduce(best == least ? best_j : 0x7fffffff, 0x7fffffff, [](int a, int b) { return min(a, b); });
    best = least;
    if ((threadIdx.x & 63) == 0 && i < n) {
        delta[(int64_t)img * n + i] = best;                  // +inf when no candidate
        parent[(int64_t)img * n + i] = best_j == 0x7fffffff ? -1 : best_j;
    }
}

// Steps 3-4 of Alg. 2 for one image per workgroup.
__global__ __launch_bounds__(SEL_THREADS) void vic_label_kernel(const float* __restrict__ rho,
                                                                const float* __restrict__ delta,
                                                                const int32_t* __restrict__ parent,
                                                                int n, int n_centers,
                                                                int32_t* __restrict__ labels,
                                                                int32_t* __restrict__ n_clusters,
                                                                int64_t batch_stride) {
    extern __shared__ __attribute__((aligned(16))) unsigned vic_lds[];
    __shared__ SelectShared sh;
    __shared__ int wave_tot[SEL_THREADS / 64];
    const int tid = threadIdx.x, b = blockIdx.x;
    rho += b * batch_stride;
    delta += b * batch_stride;
    parent += b * batch_stride;
    labels += b * batch_stride;
    unsigned* keys = vic_lds;                          // [n]  order-preserving keys of gamma, later root pointers
    int32_t* chosen = reinterpret_cast<int32_t*>(vic_lds + n);     // [n_centers] centre indices, later cluster ids [n]
    int32_t* cid = reinterpret_cast<int32_t*>(vic_lds + n);        // (reuses `chosen` once the roots are marked)
    unsigned* is_root = vic_lds + 2 * (size_t)n;       // [n]

    // largest gamma = rho delta first (+inf without a parent): complement of the bit pattern (gamma >= 0)
    for (int i = tid; i < n; i += SEL_THREADS)
        keys[i] = ~__float_as_uint(parent[i] < 0 ? INFINITY : rho[i] * delta[i]);
    block_select_emit(keys, n, n_centers, chosen, 0, sh);
    __syncthreads();
    for (int i = tid; i < n; i += SEL_THREADS) is_root[i] = parent[i] < 0 ? 1u : 0u;
    __syncthreads();
    for (int r = tid; r < n_centers; r += SEL_THREADS) is_root[chosen[r]] = 1u;
    __syncthreads();

    // cluster id of a root = number of roots with a lower index (block-wide exclusive scan over
    // chunks of SEL_THREADS tokens), and the pointer every token starts from
    const int running = block_exclusive_scan<SEL_THREADS>(
        0, n, wave_tot, [&](int i) { return (int)is_root[i]; },
        [&](int i, int f, int before) {
            cid[i] = before;
            keys[i] = f ? (unsigned)i : (unsigned)parent[i];
        });
    if (tid == 0) n_clusters[b] = (int32_t)running;

    // pointer jumping: after at most ceil(log2 n) rounds every pointer is a root, which points at itself; chains of
    // parents are short, so the rounds end with the first that moves nothing
    for (int span = 1; span < n; span <<= 1) {
        bool moved = false;
        for (int i = tid; i < n; i += SEL_THREADS) {
            const unsigned p = keys[i], q = keys[p];
            keys[i] = q;                // concurrent updates only move a pointer further up its own chain
            moved |= q != p;
        }
        if (!__syncthreads_or(moved)) break;
    }
    for (int i = tid; i < n; i += SEL_THREADS) labels[i] = cid[keys[i]];
}

size_t vic_workspace_bytes(int B, int n) {
    const size_t n_pad = ((size_t)n + 3) / 4 * 4;
    // per image: inner products, squared norms (two halves, one padded), rho, delta, parent
    return (size_t)B * (up256(n_pad * n * 4) + up256(n_pad * 4) + 4 * up256((size_t)n * 4));
}

int launch_vic(const uint16_t* feats, int64_t row_stride, int64_t batch_stride, const float* pos, int B,
               int n, int D, float d_c, float tau, int n_centers, int32_t* labels, int32_t* n_clusters,
               float* rho_out, float* delta_out, int32_t* parent_out, float* dist_out, void* ws,
               hipStream_t s) {
    if (B == 0) return VITCOP_OK;
    if (n == 0) {
        hipLaunchKernelGGL(vic_label_kernel, dim3(B), dim3(SEL_THREADS), 16, s, nullptr, nullptr, nullptr, 0, 0, labels,
                           n_clusters, 0);
        return launch_status("vic_label");
    }
    const int64_t n_pad = ((int64_t)n + 3) / 4 * 4;
    char* p = static_cast<char*>(ws);
    auto take = [&](size_t bytes) {
        char* r = p;
        p += up256(bytes);
        return r;
    };
    float* gram = reinterpret_cast<float*>(take((size_t)B * n_pad * n * 4));
    float* sq = reinterpret_cast<float*>(take((size_t)B * n_pad * 4));
    float* rho_ws = reinterpret_cast<float*>(take((size_t)B * n * 4));
    float* delta_ws = reinterpret_cast<float*>(take((size_t)B * n * 4));
    float* sq2 = reinterpret_cast<float*>(take((size_t)B * n * 4));
    int32_t* parent_ws = reinterpret_cast<int32_t*>(take((size_t)B * n * 4));
    float* rho = rho_out ? rho_out : rho_ws;
    float* delta = delta_out ? delta_out : delta_ws;
    int32_t* parent = parent_out ? parent_out : parent_ws;

    const dim3 row_grid((unsigned)((int64_t)((n + VIC_ROWS - 1) / VIC_ROWS) * B));
    const float c = -1.4426950408889634f / (d_c * d_c);
    const int64_t batch = (int64_t)n * n_pad;
    int rc = launch_gram(feats, row_stride, batch_stride, sq, n, sq2 - sq, gram, n_pad, batch, n, D, B, s);
    if (rc) return rc;
    hipLaunchKernelGGL(vic_density_kernel, row_grid, dim3(VIC_THREADS), 0, s, gram, n_pad, batch, sq, n, sq2 - sq, n, c, rho,
                       dist_out);
    rc = launch_status("vic_density");
    if (rc) return rc;
    hipLaunchKernelGGL(vic_parent_kernel, row_grid, dim3(VIC_THREADS), 0, s, gram, n_pad, batch, sq, n, sq2 - sq, pos, rho, n,
                       tau * tau, delta, parent);
    rc = launch_status("vic_parent");
    if (rc) return rc;
    const size_t lds = (size_t)3 * n * 4 + 16;
    static std::atomic<bool> attr_set{false};   // set once; a second thread repeating the call is harmless
    if (!attr_set.load(std::memory_order_acquire)) {
        rc = hip_status(hipFuncSetAttribute((const void*)vic_label_kernel,
                                            hipFuncAttributeMaxDynamicSharedMemorySize,
                                            3 * VITCOP_VIC_MAX_TOKENS * 4 + 16),
                        "hipFuncSetAttribute(vic_label)");
        if (rc) return rc;
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(vic_label_kernel, dim3(B), dim3(SEL_THREADS), lds, s, rho, delta, parent, n, n_centers, labels,
                       n_clusters, (int64_t)n);
    return launch_status("vic_label");
}

}  // namespace vitcop
