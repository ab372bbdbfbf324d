// Internal declarations shared by the translation units of libvitcop.
// Host-side argument checking lives in api.cpp; each *.hip file owns its
// kernels and exposes one or two launch functions declared here.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "vitcop.h"

namespace vitcop {

static inline size_t up256(size_t n) { return (n + 255) & ~(size_t)255; }

// Records a thread-local message and returns `code` (a VITCOP_E* value).
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
// VITCOP_OK, or records the HIP error text and returns VITCOP_EHIP.
int hip_status(hipError_t e, const char* what);
int launch_status(const char* kernel_name);

// ---- K-norm + selection (knorm_select.hip) -------------------------------
int launch_knorm(const uint16_t* k, int64_t row_stride, int64_t batch_stride, int B,
                 int row_elems, int vis_start, int n_vis, float* norms, hipStream_t s);
// Ranks the n_vis candidates of each sample and writes the keep list.
// value(b,i) = sum_{p<n_parts} parts[p*part_stride + b*sample_stride + offset + i];
// do_sqrt: rank sqrt(value); norms_out (nullable) receives the ranked values.
int launch_select_smallest(const float* parts, int n_parts, int64_t part_stride,
                           int64_t sample_stride, int64_t offset, int do_sqrt,
                           float* norms_out, int B, int T, int vis_start, int n_vis,
                           int keep, int32_t* keep_idx, hipStream_t s,
                           const int32_t* n_vis_samples = nullptr, int32_t* n_vis_samples_out = nullptr);

// ---- compaction (compact.hip) --------------------------------------------
int launch_compact(const vitcop_gather_t* t, int n, const int32_t* idx, int B, int T_out,
                   hipStream_t s);

// ---- Stage I filter (filter.hip) -----------------------------------------
int launch_filter(const uint16_t* q_cls, const uint16_t* k, int B, int N, int H, int d,
                  int keep, float scale, float* scores_out, int32_t* idx_out,
                  float* logits_ws, hipStream_t s);
// Device address of the library-owned scratch array of FILTER_STATIC_SCRATCH_BYTES on the current device.
constexpr size_t FILTER_STATIC_SCRATCH_BYTES = VITCOP_FILTER_STATIC_MAX_BYTES;
int filter_static_scratch(float** out);

// ---- attention (attn.hip) -------------------------------------------------
// kv_batch: elements between two samples' K and V (0: dense, N * Hkv * d)
int launch_attn(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out,
                float* lse, int B, int N, int Hq, int Hkv, int d, float scale, int causal,
                hipStream_t s, int64_t kv_batch = 0);

// ---- projection GEMM (gemm.hip) -------------------------------------------
int gemm_sumsq_parts(int N);
int launch_gemm(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y,
                int64_t y_stride, const uint16_t* res, int64_t res_stride, int M, int N,
                int K, float* sumsq_parts, hipStream_t s);
// y1 = x W1^T [M,N1] and y2 = x W2^T [M,N2] (dense outputs), one launch when the shapes allow
int launch_gemm_pair(const uint16_t* x, int64_t x_stride, const uint16_t* w1, uint16_t* y1, int N1,
                     const uint16_t* w2, uint16_t* y2, int N2, int M, int K, hipStream_t s);

// The same two calls with a scratch buffer: launches of at most 256 rows (gemm_skinny.hip) and, where that is
// estimated faster, of at most 1536 then go out as k-slices whose fp32 partials live in `ws`; with ws == nullptr, too
// small a buffer or any other shape they are the calls above.  gemm_workspace_bytes is what a cut of one launch
// (N = N1 + N2 for a pair) may need, also where whole tiles are taken in the end; 0 where none is considered.
size_t gemm_workspace_bytes(int M, int N, int K);
int launch_gemm_ws(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y, int64_t y_stride,
                   const uint16_t* res, int64_t res_stride, int M, int N, int K, float* sumsq_parts, void* ws,
                   size_t ws_bytes, hipStream_t s);
// y = x W^T + res as launch_gemm_ws, and norm_out = RMSNorm(y) * ln_w (rows norm_stride apart): fused
// into the few-row path's reduction where that applies, otherwise the projection and launch_rmsnorm.
int launch_gemm_norm_ws(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y, int64_t y_stride,
                        const uint16_t* res, int64_t res_stride, int M, int N, int K, const uint16_t* ln_w,
                        float eps, uint16_t* norm_out, int64_t norm_stride, void* ws, size_t ws_bytes,
                        hipStream_t s);
// Three projections of the same input (dense outputs [M, n[i]]), n[0] and n[1] multiples of 128: one launch on the
// few-row path, and of whole tiles above 1024 rows where that is no slower; otherwise the first alone and the other two
// as a pair.
int launch_gemm_triple_ws(const uint16_t* x, int64_t x_stride, const uint16_t* const w[3], uint16_t* const y[3],
                          const int n[3], int M, int K, void* ws, size_t ws_bytes, hipStream_t s);
// out = silu(x wg^T) * (x wu^T) [M, F]: one launch with the activation in the tiles' epilogue, on few rows also in the
// reduction of k-slices; otherwise the pair of projections into gate and up [M, F] and launch_silu_mul.
int launch_gemm_gated_ws(const uint16_t* x, int64_t x_stride, const uint16_t* wg, const uint16_t* wu, int F,
                         uint16_t* gate, uint16_t* up, uint16_t* out, int M, int K, void* ws, size_t ws_bytes,
                         hipStream_t s);
int launch_gemm_pair_ws(const uint16_t* x, int64_t x_stride, const uint16_t* w1, uint16_t* y1, int N1,
                        const uint16_t* w2, uint16_t* y2, int N2, int M, int K, void* ws, size_t ws_bytes,
                        hipStream_t s);
// q = x Wq^T (dense [M, Hq d]), k = x Wk^T and v = x Wv^T with the rotary embedding of q and k at positions[m]: where
// the projections leave partial sums (few rows, or split-K of K and of the Q/V pair) one launch adds them up and
// turns q and k; otherwise launch_gemm_triple_ws and rope_kernel.  Row m of k and v is row m % T of sample m / T, whose
// rows start at k_dst and v_dst + (m / T) * kv_batch (plus rows[m] rows, if given: the new tokens of a decoding step,
// T = 1, go to their caches' next rows).  k_tmp and v_tmp: scratch [M, Hkv d].
// gemm_qkv_workspace_bytes: what ws must hold for every path this may take at M rows.
// parts_out (nullable): of at most 256 rows the partial sums (columns [k | q | v]) are left for the caller to finish;
// parts_out->part == nullptr afterwards means that everything is done.
struct SkParts;
size_t gemm_qkv_workspace_bytes(int M, int Hq, int Hkv, int d, int K);
int launch_gemm_qkv_rope_ws(const uint16_t* x, int64_t x_stride, const uint16_t* wk, const uint16_t* wq,
                            const uint16_t* wv, uint16_t* k_tmp, uint16_t* q, uint16_t* v_tmp, int Hq, int Hkv, int d,
                            const int32_t* positions, float theta, int M, int K, void* ws, size_t ws_bytes,
                            uint16_t* k_dst, uint16_t* v_dst, int T, int64_t kv_batch, hipStream_t s,
                            const int32_t* rows = nullptr, SkParts* parts_out = nullptr);
// Up to three weight matrices side by side (projections of the same input in one launch): matrix i
// covers the columns [n_end[i-1], n_end[i]) of the launch (boundaries multiples of 128; unused
// entries repeat N) and writes its own output with its own row stride.
struct SkMats {
    const uint16_t* w[3];
    uint16_t* y[3];
    int64_t y_stride[3];
    int n_end[3];
};
struct SkPick {
    int mi, start;                       // matrix of a column and that matrix's first column
};
__host__ __device__ inline SkPick sk_pick(const SkMats& mats, int n) {
    const int mi = (n >= mats.n_end[0] ? 1 : 0) + (n >= mats.n_end[1] ? 1 : 0);
    return {mi, mi == 0 ? 0 : (mi == 1 ? mats.n_end[0] : mats.n_end[1])};
}
// one matrix of N columns, or with w2 a pair: w2 and y2 (row stride y2_stride, 0: y_stride) from column n_split on
inline SkMats sk_mats(const uint16_t* w, uint16_t* y, int64_t y_stride, int N, const uint16_t* w2 = nullptr,
                      uint16_t* y2 = nullptr, int n_split = 0, int64_t y2_stride = 0) {
    return SkMats{{w, w2 ? w2 : w, w}, {y, w2 ? y2 : y, y}, {y_stride, y2_stride ? y2_stride : y_stride, y_stride},
                  {w2 ? n_split : N, N, N}};
}
// The partial sums of a launch cut into k-slices: part[slice][m][n], N columns, M rows.
struct SkParts {
    const float* part;
    int slices, N, M;
};
// k, q and v of a layer (in this order) as partial sums: for each the launch it belongs to and its first
// column there.
struct QkvParts {
    SkParts parts[3];
    int col0[3];
};
// q [M, Hq d], k and v (rows as for launch_gemm_qkv_rope_ws) = the partial sums added in slice order and rounded to
// bf16, q and k then turned by the rotary embedding at positions[m] (rope_kernel's arithmetic).
int launch_qkv_finish(const QkvParts& P, uint16_t* k, uint16_t* q, uint16_t* v, int Hq, int Hkv, int d,
                      const int32_t* positions, float theta, int T, int64_t kv_stride, hipStream_t s,
                      const int32_t* kv_rows = nullptr);

int launch_partial_reduce(const SkParts& parts, int N, const SkMats& mats, const uint16_t* res, int64_t res_stride,
                          float* sumsq_parts, const uint16_t* ln_w, float eps, uint16_t* norm_out,
                          int64_t norm_stride, uint16_t* gated_out, hipStream_t s);
bool partial_reduce_fuses_norm(int N);
// The per-slice partials of a decoding attention: part_o [B*Hq][n_splits][d] unnormalised outputs, part_ml
// [B*Hq][n_splits][2] (running maximum in log2 units, sum).  With hand_over != nullptr and at most
// DECODE_PARTS_MAX_SPLITS slices launch_decode_attn leaves the combination to the caller's next kernel
// (`out` is then not written) and describes the partials there; otherwise hand_over->part_o is null.
constexpr int DECODE_PARTS_MAX_SPLITS = 16;
struct DecodeParts {
    const float* part_o;
    const float* part_ml;
    int n_splits;
};

// gemv.hip: projections of at most GV_MAX_ROWS rows as a stream over the weights (decoding steps), with
// RMSNorm of x in the prologue (ln_w != nullptr) and the residual add, silu(gate) * up, or the rotary
// embedding with the KV-cache append in the epilogue.  N even, W dense [N][K], K within gemv_applies.
constexpr int GV_MAX_ROWS = 4;
bool gemv_applies(int B, int K);
int launch_gemv(const uint16_t* x, int64_t x_stride, const uint16_t* ln_w, float eps, const uint16_t* w, uint16_t* y,
                int64_t y_stride, const uint16_t* res, int64_t res_stride, int B, int N, int K, hipStream_t s,
                const DecodeParts* attn = nullptr, int head_dim = 0);
int launch_gemv_gated(const uint16_t* x, int64_t x_stride, const uint16_t* ln_w, float eps, const uint16_t* wg,
                      const uint16_t* wu, uint16_t* act, int64_t act_stride, int B, int F, int K, hipStream_t s);
int launch_gemv_qkv_rope(const uint16_t* x, int64_t x_stride, const uint16_t* ln_w, float eps, const uint16_t* wq,
                         const uint16_t* wk, const uint16_t* wv, uint16_t* q, uint16_t* k_dst, uint16_t* v_dst,
                         int64_t kv_batch, const int32_t* positions, int B, int Hq, int Hkv, int d, int K, float theta,
                         hipStream_t s, const int32_t* kv_rows = nullptr);

size_t gemm_skinny_workspace_bytes(int M, int N, int K);
bool gemm_skinny_fuses_norm(int M, int N, int K);
int launch_gemm_skinny_gated(const uint16_t* x, int64_t x_stride, const uint16_t* wg, const uint16_t* wu, int F,
                             uint16_t* out, int M, int K, void* ws, hipStream_t s);
// (parts_out != nullptr: the rows are left as partial sums, described there, for the caller to finish;
// parts_out->part == nullptr afterwards means the launch wrote its outputs directly.)
int launch_gemm_skinny3(const uint16_t* x, int64_t x_stride, const uint16_t* const w[3], uint16_t* const y[3],
                        const int n[3], int M, int K, void* ws, hipStream_t s, SkParts* parts_out = nullptr);
int launch_gemm_skinny(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y, int64_t y_stride,
                       const uint16_t* res, int64_t res_stride, int M, int N, int K, float* sumsq_parts,
                       const uint16_t* w2, uint16_t* y2, int n_split, void* ws, hipStream_t s,
                       const uint16_t* ln_w = nullptr, float eps = 0.f, uint16_t* norm_out = nullptr,
                       int64_t norm_stride = 0);

// gram[b][i][j] + gram[b][j][i] = <f_i, f_j> (fp32, i != j) between the rows of each of `batch` matrices, from MFMA, and
// sq[b][i] + (sq + sq_half)[b][i] = <f_i, f_i>; rows of gram writable up to the next multiple of 4 entries,
// gram_stride % 4 == 0
int launch_gram(const uint16_t* f, int64_t row_stride, int64_t batch_stride, float* sq, int64_t sq_batch, int64_t sq_half,
                float* gram, int64_t gram_stride, int64_t gram_batch, int n, int K, int batch, hipStream_t s);

// ---- Visual Information Clustering (vic.hip) --------------------------------
size_t vic_workspace_bytes(int B, int n);
int launch_vic(const uint16_t* feats, int64_t row_stride, int64_t batch_stride, const float* pos, int B,
               int n, int D, float d_c, float tau, int n_centers, int32_t* labels, int32_t* n_clusters,
               float* rho_out, float* delta_out, int32_t* parent_out, float* dist_out, void* ws,
               hipStream_t s);

// ---- collaborative pruning and merging (collab.hip) -------------------------
size_t collab_workspace_bytes(int B, int n);
int launch_collab(const uint16_t* feats, int64_t row_stride, int64_t batch_stride, const int32_t* labels,
                  const int32_t* n_clusters, const float* norms, int B, int n, int D, int budget,
                  uint16_t* out_feats, int32_t* out_index, int32_t* n_out, int32_t* assign, void* ws,
                  hipStream_t s);

// ---- decoder-layer pieces (decoder.hip) -------------------------------------
int launch_rmsnorm(const uint16_t* x, int64_t x_stride, const uint16_t* w, float eps, uint16_t* y,
                   int64_t y_stride, int M, int D, hipStream_t s);
// in place; q [n_tokens,Hq,d] and k [n_tokens,Hkv,d] (either may be null), positions [n_tokens]
int launch_rope(uint16_t* q, uint16_t* k, const int32_t* positions, int64_t n_tokens, int Hq, int Hkv, int d,
                float theta, hipStream_t s);
// q embedded in place, k embedded on its way from k [n_tokens,Hkv,d] to k_dst, v (nullable) copied to v_dst: token m is
// row m % T of sample m / T, whose rows start kv_batch elements after the sample before (rows, nullable: rows[m] further on)
int launch_rope_append(uint16_t* q, const uint16_t* k, const uint16_t* v, const int32_t* positions, int64_t n_tokens,
                       int Hq, int Hkv, int d, float theta, uint16_t* k_dst, uint16_t* v_dst, int64_t T,
                       int64_t kv_batch, hipStream_t s, const int32_t* rows = nullptr);
int launch_silu_mul(const uint16_t* gate, const uint16_t* up, uint16_t* out, int64_t n_elems, hipStream_t s);

// ---- decoding step over the KV cache (decode.hip) ---------------------------
size_t decode_workspace_bytes(int B, int N, int Hq, int Hkv, int d);
// The new tokens' k, q and v as partial sums of their projections (columns [k | q | v] of `parts`, row b for sample b): the
// attention adds them up as launch_qkv_finish does, turns q and k, and appends k and v to the caches as the last row that
// it attends over.
struct DecodeNew {
    SkParts parts;                       // parts.part == nullptr: q is given, and the caches hold the new rows
    const int32_t* positions;            // [B]
    float rope_c;                        // -2 log2(theta) / d
    uint16_t *k, *v;                     // the caches, for writing
};
// kv_batch: elements between two samples' caches (0: dense, N * Hkv * d); n_cached_samples (nullable, device
// [B]): sample b attends over its first n_cached_samples[b] + 1 <= N rows only; fresh (nullable): instead of q
int launch_decode_attn(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out, float* lse, int B,
                       int N, int Hq, int Hkv, int d, float scale, void* ws, hipStream_t s, int64_t kv_batch = 0,
                       DecodeParts* hand_over = nullptr, const int32_t* n_cached_samples = nullptr,
                       const DecodeNew* fresh = nullptr);

}  // namespace vitcop
