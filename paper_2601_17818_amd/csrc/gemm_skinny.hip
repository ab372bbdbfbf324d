// Linear projections y = x W^T for FEW rows (M <= 256): what the projections of a decoder layer
// look like after the pruning of Sec. 3.2.2 has cut the sequence to a few hundred tokens.  The
// weight matrix is then nearly all of the traffic (one pass over W per launch) and the launch is
// bound by HBM, not by the matrix cores, so all 256 CUs must stream whatever N and K are:
//
//   * one tile holds all rows of x (32 to 256 in steps of 32) and 64, 96 or 128 columns, and the
//     k-range is cut into slices until about 256 workgroups exist (gemm_kernel.h; its ring of
//     direct loads keeps three k-steps of both operands in flight per workgroup);
//   * up to three weight matrices can sit side by side in one launch (K, Q and V; gate and up);
//   * the slices leave fp32 partial sums; a second kernel adds them in slice order (deterministic)
//     and finishes the rows in one of three ways: residual, bf16 rounding and, for the K projection,
//     the per-128-column sums of squares of the rounded outputs for the K-norm of Eq. 4; the same
//     plus the RMSNorm of the finished row; or the gated activation silu(gate) * up of the MLP.
//     The same reductions serve the k-slices of launches with more rows (gemm.hip);
//   * the MLP's gate and up projections need no partial sums where their columns alone keep most
//     CUs streaming: the activation is then applied in the tile's epilogue.
#include <algorithm>
#include <cmath>
#include "gemm_kernel.h"
#include "gemm_plan.h"

namespace vitcop {

// The sum, in slice order, of the partials of row m, columns n .. n+8 (n a multiple of 8).  The first four slices'
// loads go out when it is declared, so that a kernel's other loads can follow before the first wait (a reduction of a few
// rows is a chain of round trips to memory); further slices follow four at a time.
struct SkSum {
    const float* p;
    int64_t slice;
    int slices;
    f32x4 a[4], b[4];
    __device__ __forceinline__ SkSum() {}
    __device__ __forceinline__ SkSum(const SkParts& P, int m, int n)
        : p(P.part + (int64_t)m * P.N + n), slice((int64_t)P.M * P.N), slices(P.slices) {
        request(0);
    }
    __device__ __forceinline__ void request(int s0) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (s0 + t < slices) {
                a[t] = *reinterpret_cast<const f32x4*>(p + (s0 + t) * slice);
                b[t] = *reinterpret_cast<const f32x4*>(p + (s0 + t) * slice + 4);
            }
    }
    __device__ __forceinline__ void add_up(float (&v)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.f;
        for (int s0 = 0; s0 < slices; s0 += 4) {
            if (s0 > 0) request(s0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (s0 + t < slices)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] += a[t][e];
                        v[4 + e] += b[t][e];
                    }
        }
    }
};

// y[m, n..n+8) = bf16(sum of the slices' partials, in slice order, + residual);
// one thread per 8 columns, 16 consecutive lanes per 128-column group, which also yields that
// group's sum of squares of the rounded outputs.
__global__ __launch_bounds__(256) void gemm_skinny_reduce_kernel(
    SkParts parts, int N, SkMats mats, const uint16_t* __restrict__ res, int64_t res_stride,
    float* __restrict__ sumsq_parts) {
    const int M = parts.M;
    const int groups = (N + SK_COLS - 1) / SK_COLS, chunks = groups * 16;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int m = (int)(id / chunks), c = (int)(id % chunks);
    const int n = c * 8, grp = c >> 4;
    float ss = 0.f;
    if (m < M && n < N) {
        SkSum sum(parts, m, n);
        uint4 r = make_uint4(0, 0, 0, 0);
        if (res) r = *reinterpret_cast<const uint4*>(res + (int64_t)m * res_stride + n);
        const SkPick pick = sk_pick(mats, n);
        uint16_t* dst = mats.y[pick.mi] + (int64_t)m * mats.y_stride[pick.mi] + (n - pick.start);
        float v[8];
        sum.add_up(v);
        if (res) {
            v[0] += bf16_lo(r.x); v[1] += bf16_hi(r.x);
            v[2] += bf16_lo(r.y); v[3] += bf16_hi(r.y);
            v[4] += bf16_lo(r.z); v[5] += bf16_hi(r.z);
            v[6] += bf16_lo(r.w); v[7] += bf16_hi(r.w);
        }
        uint4 o;
        o.x = pack_bf16(v[0], v[1]);
        o.y = pack_bf16(v[2], v[3]);
        o.z = pack_bf16(v[4], v[5]);
        o.w = pack_bf16(v[6], v[7]);
        *reinterpret_cast<uint4*>(dst) = o;
        if (sumsq_parts) {
            float a;
            a = bf16_lo(o.x); ss = fmaf(a, a, ss);
            a = bf16_hi(o.x); ss = fmaf(a, a, ss);
            a = bf16_lo(o.y); ss = fmaf(a, a, ss);
            a = bf16_hi(o.y); ss = fmaf(a, a, ss);
            a = bf16_lo(o.z); ss = fmaf(a, a, ss);
            a = bf16_hi(o.z); ss = fmaf(a, a, ss);
            a = bf16_lo(o.w); ss = fmaf(a, a, ss);
            a = bf16_hi(o.w); ss = fmaf(a, a, ss);
        }
    }
    if (sumsq_parts) {                                   // uniform branch: every lane takes part in the shuffles
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
        if ((c & 15) == 0 && m < M && n < N) sumsq_parts[(int64_t)grp * M + m] = ss;
    }
}

// The same reduction followed by an RMSNorm of the finished row (the next operation of a decoder
// layer after its attention and MLP output projections): y as above, and
// norm_out[m, :] = y[m, :] / sqrt(mean(y[m, :]^2) + eps) * ln_w, computed from the ROUNDED y exactly as
// rmsnorm_kernel does.  One workgroup per row; a thread owns the chunks tid, tid + THREADS, ... (J of them).
// Everything a thread reads is requested before the first wait (half the threads, two chunks each one after the other, the
// residual and the weight when they were needed: 4096 columns in four slices, 317 rows 6.95 -> 6.70 us, 115 rows
// 5.10 -> 4.79, 64 rows 4.75 either way; the plain reduction of 640 rows 6.5 -> 6.05, of 93 rows x 8192 5.0 -> 4.35).
// Rows of fewer chunks take fewer threads: 384 idle ones of 512 cost a layer of 1024 columns half a per cent.
constexpr int SK_NORM_THREADS = 512, SK_NORM_CHUNKS = 8;         // at most

template <int THREADS, int J>
__global__ __launch_bounds__(THREADS) void gemm_skinny_reduce_norm_kernel(
    SkParts parts, int N, uint16_t* __restrict__ y, int64_t y_stride, const uint16_t* __restrict__ res,
    int64_t res_stride, const uint16_t* __restrict__ ln_w, float eps, uint16_t* __restrict__ norm_out,
    int64_t norm_stride) {
    constexpr int AHEAD = J < 2 ? J : 2;             // chunks requested together
    __shared__ float wave_part[THREADS / 64];
    const int m = blockIdx.x, tid = threadIdx.x;
    const int chunks = N / 8;
    u32x4 held[J], weight[J];            // (native vector types: arrays of the uint4 struct end up in scratch)
    float ss = 0.f;
#pragma unroll
    for (int j0 = 0; j0 < J; j0 += AHEAD) {
        SkSum sum[AHEAD];
        u32x4 r[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int c = tid + THREADS * (j0 + u);
            if (c >= chunks) continue;
            sum[u] = SkSum(parts, m, 8 * c);
            r[u] = res ? *reinterpret_cast<const u32x4*>(res + (int64_t)m * res_stride + 8 * c) : u32x4{0, 0, 0, 0};
            weight[j0 + u] = *reinterpret_cast<const u32x4*>(ln_w + 8 * c);
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int c = tid + THREADS * (j0 + u);
            if (c >= chunks) continue;
            float v[8];
            sum[u].add_up(v);
            if (res)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[2 * e] += bf16_lo(r[u][e]);
                    v[2 * e + 1] += bf16_hi(r[u][e]);
                }
            const u32x4 o = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7])};
            *reinterpret_cast<u32x4*>(y + (int64_t)m * y_stride + 8 * c) = o;
            held[j0 + u] = o;
            ss = sumsq8(make_uint4(o.x, o.y, o.z, o.w), ss);
        }
    }
    ss = wave_sum(ss);
    if ((tid & 63) == 0) wave_part[tid >> 6] = ss;
    __syncthreads();
    ss = 0.f;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) ss += wave_part[w];
    const float r = __builtin_amdgcn_rsqf(ss / (float)N + eps);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int c = tid + THREADS * j;
        if (c >= chunks) continue;
        const u32x4 v = held[j], g = weight[j];
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = pack_bf16(bf16_lo(v[e]) * r * bf16_lo(g[e]), bf16_hi(v[e]) * r * bf16_hi(g[e]));
        *reinterpret_cast<u32x4*>(norm_out + (int64_t)m * norm_stride + 8 * c) = o;
    }
}

// The reduction of a gate/up pair launch (columns [0, F) gate, [F, 2F) up) followed by the gated
// activation of the MLP: out[m, n] = bf16(silu(g) * u) with g and u the bf16-rounded projections,
// exactly what silu_mul_kernel computes from stored gate and up tensors.  One thread per 8 columns.
__global__ __launch_bounds__(256) void gemm_skinny_reduce_silu_kernel(
    SkParts parts, int F, uint16_t* __restrict__ out, int64_t out_stride) {
    const int chunks = F / 8, M = parts.M;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int m = (int)(id / chunks), c = (int)(id % chunks);
    if (m >= M) return;
    // bf16(sum of the partials of the 8 columns from n on, in slice order), packed
    auto reduced = [&](SkSum& sum) {
        float v[8];
        sum.add_up(v);
        return make_uint4(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7]));
    };
    SkSum gate(parts, m, 8 * c), up(parts, m, F + 8 * c);
    const uint4 g = reduced(gate), u = reduced(up);
    auto gated = [](uint32_t gw, uint32_t uw) {
        const float g0 = bf16_lo(gw), g1 = bf16_hi(gw);
        const float s0 = g0 / (1.0f + __expf(-g0)), s1 = g1 / (1.0f + __expf(-g1));
        return pack_bf16(s0 * bf16_lo(uw), s1 * bf16_hi(uw));
    };
    *reinterpret_cast<uint4*>(out + (int64_t)m * out_stride + 8 * c) =
        make_uint4(gated(g.x, u.x), gated(g.y, u.y), gated(g.z, u.z), gated(g.w, u.w));
}

// q, k and v of a decoder layer straight from the partial sums of their projections (up to three sets of
// partials: the three matrices of one few-row launch, or K from one split-K launch and Q, V from another),
// with the rotary embedding of q and k: what the plain reductions followed by rope_kernel compute, value for
// value (sum in slice order, rounded to bf16, turned in fp32 at positions[m], rounded), in one launch.
// A thread owns 16 columns: of a q or k head the 8 low channels from 8 j on and the 8 high channels they pair
// with; of v 16 consecutive columns.  Row m is row m % T of sample m / T: k and v go to that row of the sample's
// cache (kv_stride elements from sample to sample, kv_rows[m] rows further on if given).
// The angles are computed once per row into LDS, as in rope_kernel, while the first four slices' loads are in flight
// (with eight sines and cosines per thread: 317 rows of 96 heads x 128 9.2 us, now 8.1; 64 rows 5.8 and 4.7).
constexpr int QF_THREADS = 256;
constexpr int QF_ANGLES = 704;           // rows of a workgroup x d/2: at most 256 / (3 d/16) rows

__global__ __launch_bounds__(QF_THREADS) void qkv_finish_kernel(
    QkvParts P, uint16_t* __restrict__ k, uint16_t* __restrict__ q, uint16_t* __restrict__ v, int Hq, int Hkv,
    int d, const int32_t* __restrict__ positions, float rope_c, int T, int64_t kv_stride,
    const int32_t* __restrict__ kv_rows, int per_wg) {
    __shared__ float2 angles[QF_ANGLES];                 // [per_wg][d / 2] sine, cosine
    const int tid = threadIdx.x, g16 = d / 16, half = d / 2, M = P.parts[0].M;
    const int units = (Hq + 2 * Hkv) * g16;
    // (per_wg == 1: a row's units go to several workgroups, side by side in y)
    const int local = per_wg > 1 ? tid / units : 0;
    int unit = per_wg > 1 ? tid - local * units : (int)blockIdx.y * QF_THREADS + tid;
    const int first = blockIdx.x * per_wg, m = first + local;
    const bool live = local < per_wg && m < M && unit < units;
    int mat = 0;                                         // 0 k, 1 q, 2 v
    if (unit >= Hkv * g16) {
        unit -= Hkv * g16;
        mat = 1;
        if (unit >= Hq * g16) {
            unit -= Hq * g16;
            mat = 2;
        }
    }
    const int head = unit / g16, j = unit - head * g16;
    const int c0 = mat == 2 ? 16 * unit : head * d + 8 * j;
    const int c1 = mat == 2 ? c0 + 8 : c0 + half;
    const SkParts& parts = mat == 0 ? P.parts[0] : (mat == 1 ? P.parts[1] : P.parts[2]);
    const int col0 = mat == 0 ? P.col0[0] : (mat == 1 ? P.col0[1] : P.col0[2]);
    const int slices = live ? parts.slices : 0;
    const int64_t slice = (int64_t)parts.M * parts.N;
    const float* p0 = parts.part + (int64_t)m * parts.N + col0 + c0;
    const int delta = c1 - c0;
    float4 w[4][4];                                      // the next four slices: both chunks of eight columns
    auto load4 = [&](int s0) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (s0 + t < slices) {
                const float* p = p0 + (s0 + t) * slice;
                w[t][0] = *reinterpret_cast<const float4*>(p);
                w[t][1] = *reinterpret_cast<const float4*>(p + 4);
                w[t][2] = *reinterpret_cast<const float4*>(p + delta);
                w[t][3] = *reinterpret_cast<const float4*>(p + delta + 4);
            }
    };
    load4(0);
    for (int i = tid; i < per_wg * half; i += QF_THREADS) {
        const int t = i / half;
        if (first + t < M) {
            const float inv_freq = __builtin_exp2f((float)(i - t * half) * rope_c);
            float sn, cs;
            sincosf((float)positions[first + t] * inv_freq, &sn, &cs);
            angles[i] = make_float2(sn, cs);
        }
    }
    float a[8], b[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = b[e] = 0.f;
    for (int s0 = 0; s0 < slices; s0 += 4) {
        if (s0 > 0) load4(s0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (s0 + t < slices) {
                a[0] += w[t][0].x; a[1] += w[t][0].y; a[2] += w[t][0].z; a[3] += w[t][0].w;
                a[4] += w[t][1].x; a[5] += w[t][1].y; a[6] += w[t][1].z; a[7] += w[t][1].w;
                b[0] += w[t][2].x; b[1] += w[t][2].y; b[2] += w[t][2].z; b[3] += w[t][2].w;
                b[4] += w[t][3].x; b[5] += w[t][3].y; b[6] += w[t][3].z; b[7] += w[t][3].w;
            }
    }
    __syncthreads();
    if (!live) return;
    uint32_t lw[4], hw[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        lw[p] = pack_bf16(a[2 * p], a[2 * p + 1]);
        hw[p] = pack_bf16(b[2 * p], b[2 * p + 1]);
    }
    uint16_t* dst = q + (int64_t)m * Hq * d;
    if (mat != 1) {
        const int sample = m / T, row = m - sample * T + (kv_rows ? kv_rows[m] : 0);
        dst = (mat == 0 ? k : v) + sample * kv_stride + (int64_t)row * Hkv * d;
    }
    if (mat != 2) {
        const float2* sc = angles + local * half + 8 * j;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            float rl[2], rh[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float sn = sc[2 * p + e].x, cs = sc[2 * p + e].y;
                const float lo = e ? bf16_hi(lw[p]) : bf16_lo(lw[p]);
                const float hi = e ? bf16_hi(hw[p]) : bf16_lo(hw[p]);
                rl[e] = lo * cs - hi * sn;
                rh[e] = hi * cs + lo * sn;
            }
            lw[p] = pack_bf16(rl[0], rl[1]);
            hw[p] = pack_bf16(rh[0], rh[1]);
        }
    }
    *reinterpret_cast<uint4*>(dst + c0) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
    *reinterpret_cast<uint4*>(dst + c1) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
}

int launch_qkv_finish(const QkvParts& P, uint16_t* k, uint16_t* q, uint16_t* v, int Hq, int Hkv, int d,
                      const int32_t* positions, float theta, int T, int64_t kv_stride, hipStream_t s,
                      const int32_t* kv_rows) {
    const int M = P.parts[0].M, units = (Hq + 2 * Hkv) * (d / 16);
    if (M == 0 || units == 0) return VITCOP_OK;
    const int per_wg = std::max(1, QF_THREADS / units);
    hipLaunchKernelGGL(qkv_finish_kernel, dim3((M + per_wg - 1) / per_wg, (units + QF_THREADS - 1) / QF_THREADS),
                       dim3(QF_THREADS), 0, s, P, k, q, v, Hq, Hkv, d, positions, -2.0f * std::log2(theta) / (float)d, T,
                       kv_stride, kv_rows, per_wg);
    return launch_status("qkv_finish");
}

size_t gemm_skinny_workspace_bytes(int M, int N, int K) {
    if (!gemm_skinny_applies(M, N, K)) return 0;
    return up256((size_t)skinny_scratch_columns(N, K) * M * 4);
}

template <int BM>
static int launch_skinny_parts(int cols, int slices, const uint16_t* x, int64_t x_stride, const SkMats& mats, int M,
                               int N, int K, float* part, hipStream_t s) {
#define VITCOP_SKINNY(BN)                                                                                            \
    return launch_gemm_cfg<BM, BN, 2, 2, GM_EPI_PART, true>(x, x_stride, mats, nullptr, 0, M, N, K, nullptr, s, K, part, N, \
                                                      slices, 0, 0, (int64_t)M * N)
    if (cols == 64) VITCOP_SKINNY(64);
    if (cols == 96) VITCOP_SKINNY(96);
    VITCOP_SKINNY(128);
#undef VITCOP_SKINNY
}
template <int BM>
static int launch_skinny_gate_up(int cols, const uint16_t* x, int64_t x_stride, const SkMats& mats, int M, int F, int K,
                                 hipStream_t s) {
    if (cols == 64)
        return launch_gemm_cfg<BM, 64, 2, 2, GM_EPI_GATED, true>(x, x_stride, mats, nullptr, 0, M, F, K, nullptr, s);
    if (cols == 96)
        return launch_gemm_cfg<BM, 96, 2, 2, GM_EPI_GATED, true>(x, x_stride, mats, nullptr, 0, M, F, K, nullptr, s);
    return launch_gemm_cfg<BM, 128, 2, 2, GM_EPI_GATED, true>(x, x_stride, mats, nullptr, 0, M, F, K, nullptr, s);
}
// f<BM>(args...) for the tile that holds M rows
#define VITCOP_BY_ROWS(f, M, ...)                  \
    switch (skinny_rows(M)) {                      \
        case 32: return f<32>(__VA_ARGS__);        \
        case 64: return f<64>(__VA_ARGS__);        \
        case 96: return f<96>(__VA_ARGS__);        \
        case 128: return f<128>(__VA_ARGS__);      \
        case 160: return f<160>(__VA_ARGS__);      \
        case 192: return f<192>(__VA_ARGS__);      \
        case 224: return f<224>(__VA_ARGS__);      \
        default: return f<256>(__VA_ARGS__);       \
    }
static int launch_skinny_slices(const SkinnyPlan& p, const uint16_t* x, int64_t x_stride, const SkMats& mats, int M,
                               int N, int K, float* part, hipStream_t s) {
    VITCOP_BY_ROWS(launch_skinny_parts, M, p.cols, p.slices, x, x_stride, mats, M, N, K, part, s)
}
static int launch_skinny_gate_up(int cols, const uint16_t* x, int64_t x_stride, const SkMats& mats, int M, int F, int K,
                                 hipStream_t s) {
    VITCOP_BY_ROWS(launch_skinny_gate_up, M, cols, x, x_stride, mats, M, F, K, s)
}
template <int BM>
static int launch_skinny_whole(const uint16_t* x, int64_t x_stride, const SkMats& mats, const uint16_t* res,
                               int64_t res_stride, int M, int N, int K, hipStream_t s) {
    return launch_gemm_cfg<BM, 128, 2, 2, GM_EPI_BF16>(x, x_stride, mats, res, res_stride, M, N, K, nullptr, s);
}
static int launch_skinny_whole(const uint16_t* x, int64_t x_stride, const SkMats& mats, const uint16_t* res,
                               int64_t res_stride, int M, int N, int K, hipStream_t s) {
    VITCOP_BY_ROWS(launch_skinny_whole, M, x, x_stride, mats, res, res_stride, M, N, K, s)
}
#undef VITCOP_BY_ROWS

bool gemm_skinny_fuses_norm(int M, int N, int K) {
    return gemm_skinny_applies(M, N, K) && !skinny_direct(N, false) && partial_reduce_fuses_norm(N);
}

// Adds up the partial sums of a launch and finishes the rows: plain (+ residual, + norm side output),
// with the RMSNorm of the finished row (ln_w), or as the gated MLP activation (gated_out; N = 2 F).
int launch_partial_reduce(const SkParts& parts, int N, const SkMats& mats, const uint16_t* res, int64_t res_stride,
                          float* sumsq_parts, const uint16_t* ln_w, float eps, uint16_t* norm_out,
                          int64_t norm_stride, uint16_t* gated_out, hipStream_t s) {
    const int M = parts.M;
    if (gated_out != nullptr) {                  // gate and up side by side
        const int64_t threads = (int64_t)M * (N / 16);
        hipLaunchKernelGGL(gemm_skinny_reduce_silu_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s,
                           parts, N / 2, gated_out, (int64_t)(N / 2));
        return launch_status("gemm_skinny_reduce_silu");
    }
    if (ln_w != nullptr) {
#define VITCOP_REDUCE_NORM(T, J)                                                                                       \
    hipLaunchKernelGGL((gemm_skinny_reduce_norm_kernel<T, J>), dim3(M), dim3(T), 0, s, parts, N, mats.y[0], mats.y_stride[0], \
                       res, res_stride, ln_w, eps, norm_out, norm_stride)
        const int chunks = N / 8;
        if (chunks <= 128) VITCOP_REDUCE_NORM(128, 1);
        else if (chunks <= 256) VITCOP_REDUCE_NORM(256, 1);
        else if (chunks <= SK_NORM_THREADS) VITCOP_REDUCE_NORM(SK_NORM_THREADS, 1);
        else if (chunks <= 2 * SK_NORM_THREADS) VITCOP_REDUCE_NORM(SK_NORM_THREADS, 2);
        else VITCOP_REDUCE_NORM(SK_NORM_THREADS, SK_NORM_CHUNKS);
#undef VITCOP_REDUCE_NORM
        return launch_status("gemm_skinny_reduce_norm");
    }
    const int chunks = (N + SK_COLS - 1) / SK_COLS * 16;
    const int64_t threads = (int64_t)M * chunks;
    hipLaunchKernelGGL(gemm_skinny_reduce_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, parts, N,
                       mats, res, res_stride, sumsq_parts);
    return launch_status("gemm_skinny_reduce");
}

bool partial_reduce_fuses_norm(int N) { return N % 8 == 0 && N <= 8 * SK_NORM_THREADS * SK_NORM_CHUNKS; }

// The launch over the matrices of `mats` (N = all their columns) through partial tiles in `ws`
// (gemm_skinny_workspace_bytes).  res and sumsq_parts only with a single matrix.  With ln_w != nullptr
// (only where gemm_skinny_fuses_norm holds, one matrix, no norm side output) norm_out also receives
// RMSNorm(y) * ln_w.
static int launch_skinny_mats(const uint16_t* x, int64_t x_stride, const SkMats& mats, const uint16_t* res,
                              int64_t res_stride, int M, int N, int K, float* sumsq_parts, void* ws, hipStream_t s,
                              const uint16_t* ln_w, float eps, uint16_t* norm_out, int64_t norm_stride,
                              uint16_t* gated_out = nullptr, SkParts* parts_out = nullptr) {
    if (parts_out) parts_out->part = nullptr;
    if (gated_out == nullptr && skinny_direct(N, sumsq_parts != nullptr))
        return launch_skinny_whole(x, x_stride, mats, res, res_stride, M, N, K, s);
    const SkinnyPlan plan = skinny_plan(M, N, K);
    if (gated_out != nullptr) {
        const int F = N / 2, cols = skinny_gated_columns(plan, M, F, K);
        if (cols != 0) {
            const SkMats gate_up{{mats.w[0], mats.w[1], mats.w[1]}, {gated_out, gated_out, gated_out}, {F, F, F}, {F, F, F}};
            return launch_skinny_gate_up(cols, x, x_stride, gate_up, M, F, K, s);
        }
    }
    const SkParts parts{static_cast<float*>(ws), plan.slices, N, M};
    const int rc = launch_skinny_slices(plan, x, x_stride, mats, M, N, K, static_cast<float*>(ws), s);
    if (rc) return rc;
    if (parts_out) {                             // the caller finishes the rows itself
        *parts_out = parts;
        return VITCOP_OK;
    }
    return launch_partial_reduce(parts, N, mats, res, res_stride, sumsq_parts, ln_w, eps, norm_out, norm_stride,
                                 gated_out, s);
}

// y = x W^T (+ res) [M,N] for M <= 256.  With w2: columns [n_split, N) use w2 and go to y2, dense (n_split a
// multiple of 128).
int launch_gemm_skinny(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y, int64_t y_stride,
                       const uint16_t* res, int64_t res_stride, int M, int N, int K, float* sumsq_parts,
                       const uint16_t* w2, uint16_t* y2, int n_split, void* ws, hipStream_t s,
                       const uint16_t* ln_w, float eps, uint16_t* norm_out, int64_t norm_stride) {
    const SkMats mats = sk_mats(w, y, y_stride, N, w2, y2, n_split, w2 ? N - n_split : 0);
    return launch_skinny_mats(x, x_stride, mats, res, res_stride, M, N, K, sumsq_parts, ws, s, ln_w, eps, norm_out,
                              norm_stride);
}

// Three projections of the same input in one launch: y[i] = x w[i]^T, [M, n[i]] dense (n[0] and n[1]
// multiples of 128).
int launch_gemm_skinny3(const uint16_t* x, int64_t x_stride, const uint16_t* const w[3], uint16_t* const y[3],
                        const int n[3], int M, int K, void* ws, hipStream_t s, SkParts* parts_out) {
    SkMats mats{{w[0], w[1], w[2]}, {y[0], y[1], y[2]}, {n[0], n[1], n[2]}, {n[0], n[0] + n[1], n[0] + n[1] + n[2]}};
    return launch_skinny_mats(x, x_stride, mats, nullptr, 0, M, n[0] + n[1] + n[2], K, nullptr, ws, s, nullptr, 0.f,
                              nullptr, 0, nullptr, parts_out);
}

// out = silu(x wg^T) * (x wu^T) [M, F] (F a multiple of 128): both projections in one launch, the
// activation in its reduction.
int launch_gemm_skinny_gated(const uint16_t* x, int64_t x_stride, const uint16_t* wg, const uint16_t* wu, int F,
                             uint16_t* out, int M, int K, void* ws, hipStream_t s) {
    SkMats mats{{wg, wu, wu}, {nullptr, nullptr, nullptr}, {0, 0, 0}, {F, 2 * F, 2 * F}};
    return launch_skinny_mats(x, x_stride, mats, nullptr, 0, M, 2 * F, K, nullptr, ws, s, nullptr, 0.f, nullptr, 0,
                              out);
}

}  // namespace vitcop
