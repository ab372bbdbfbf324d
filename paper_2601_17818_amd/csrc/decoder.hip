// Element-wise and row-wise pieces of a LLaMA-family decoder layer around the pruned prefill
// (the language model of LLaVA-1.5 / LLaVA-NeXT, Sec. 4.1 of arXiv 2601.17818): RMSNorm, rotary
// position embedding with explicit (gathered) positions, and the SiLU gate of the MLP.  All
// three are single passes over their operands (HBM-bound); the matrix products between them
// are the projection kernel's.
#include "vitcop_internal.h"
#include "device_utils.h"

#include <algorithm>
#include <cmath>

namespace vitcop {

// y = x / sqrt(mean(x^2) + eps) * w.  One wavefront per row; the row is read once and kept in
// registers for D <= 8192 (16 chunks of 8 per lane), otherwise read twice.
constexpr int RN_THREADS = 256;
constexpr int RN_MAX_CHUNKS = 16;

__global__ __launch_bounds__(RN_THREADS) void rmsnorm_kernel(const uint16_t* __restrict__ x, int64_t x_stride,
                                                             const uint16_t* __restrict__ w, float eps,
                                                             uint16_t* __restrict__ y, int64_t y_stride, int M,
                                                             int D) {
    const int lane = threadIdx.x & 63;
    const int m = blockIdx.x * (RN_THREADS / 64) + (threadIdx.x >> 6);
    if (m >= M) return;
    const uint16_t* row = x + (int64_t)m * x_stride;
    uint16_t* out = y + (int64_t)m * y_stride;
    const int chunks = D / 8;                                // 16-byte chunks in the row
    u32x4 held[RN_MAX_CHUNKS];           // (a native vector type: arrays of the uint4 struct end up in scratch)
    float acc = 0.f;
    const bool fits = chunks <= 64 * RN_MAX_CHUNKS;
#pragma unroll
    for (int j = 0; j < RN_MAX_CHUNKS; ++j) {
        const int c = lane + 64 * j;
        if (c < chunks) {
            held[j] = *reinterpret_cast<const u32x4*>(row + 8 * c);
            acc = sumsq8(make_uint4(held[j].x, held[j].y, held[j].z, held[j].w), acc);
        }
    }
    for (int c = lane + 64 * RN_MAX_CHUNKS; c < chunks; c += 64)
        acc = sumsq8(*reinterpret_cast<const uint4*>(row + 8 * c), acc);
    acc = wave_sum(acc);
    const float r = __builtin_amdgcn_rsqf(acc / (float)D + eps);
    auto scale8 = [&](const uint4& v, const uint4& g) {
        uint4 o;
        o.x = pack_bf16(bf16_lo(v.x) * r * bf16_lo(g.x), bf16_hi(v.x) * r * bf16_hi(g.x));
        o.y = pack_bf16(bf16_lo(v.y) * r * bf16_lo(g.y), bf16_hi(v.y) * r * bf16_hi(g.y));
        o.z = pack_bf16(bf16_lo(v.z) * r * bf16_lo(g.z), bf16_hi(v.z) * r * bf16_hi(g.z));
        o.w = pack_bf16(bf16_lo(v.w) * r * bf16_lo(g.w), bf16_hi(v.w) * r * bf16_hi(g.w));
        return o;
    };
#pragma unroll
    for (int j = 0; j < RN_MAX_CHUNKS; ++j) {
        const int c = lane + 64 * j;
        if (c < chunks)
            *reinterpret_cast<uint4*>(out + 8 * c) = scale8(make_uint4(held[j].x, held[j].y, held[j].z, held[j].w),
                                                            *reinterpret_cast<const uint4*>(w + 8 * c));
    }
    if (!fits)
        for (int c = lane + 64 * RN_MAX_CHUNKS; c < chunks; c += 64)
            *reinterpret_cast<uint4*>(out + 8 * c) =
                scale8(*reinterpret_cast<const uint4*>(row + 8 * c), *reinterpret_cast<const uint4*>(w + 8 * c));
}

int launch_rmsnorm(const uint16_t* x, int64_t x_stride, const uint16_t* w, float eps, uint16_t* y,
                   int64_t y_stride, int M, int D, hipStream_t s) {
    if (M == 0) return VITCOP_OK;
    hipLaunchKernelGGL(rmsnorm_kernel, dim3((unsigned)((M + RN_THREADS / 64 - 1) / (RN_THREADS / 64))),
                       dim3(RN_THREADS), 0, s, x, x_stride, w, eps, y, y_stride, M, D);
    return launch_status("rmsnorm");
}

// Rotary embedding, rotate-half pairing: channel i < d/2 of a head pairs with channel i + d/2 and the pair turns by
// position * theta^(-2i/d).  A unit of work is 8 consecutive low channels of a head of q or k and the 8 high channels
// they pair with, or 8 channels of v; q is turned in place, k on its way from k to k_dst (the same rows for an embedding
// in place), v copied to v_dst.  Token m is row m % T of sample m / T, whose rows of k_dst and v_dst start kv_batch
// elements after the sample before (and rows[m] rows further on, if given).
//
// The angles depend on the token and the channel alone, so a workgroup (the units of one token, or of a few where they
// are fewer than its threads) computes them once into LDS for all heads.  Bound by its traffic from some thousand tokens
// on: 2536 tokens x 64 heads x 128 with their V, 125 MB, 24.4 us = 5.1 TB/s (eight sines and cosines per unit and two
// copies to the cache afterwards: 20.8 + 17.3 us).
constexpr int RP_THREADS = 256;
constexpr int RP_MAX_HALF = 1024;          // longer heads (none that a layer takes) compute their angles unit by unit

__global__ __launch_bounds__(RP_THREADS) void rope_kernel(
    uint16_t* __restrict__ q, const uint16_t* k, const uint16_t* __restrict__ v, const int32_t* __restrict__ positions,
    int64_t n_tokens, int Hq, int Hkv, int d, float neg_log2_theta_2_over_d, uint16_t* k_dst,
    uint16_t* __restrict__ v_dst, int64_t T, int64_t kv_batch, const int32_t* __restrict__ rows, int per_wg) {
    extern __shared__ __attribute__((aligned(16))) float2 rp_angles[];         // [per_wg][d / 2] sine, cosine
    const int tid = threadIdx.x, half = d / 2, groups = d / 16;
    const int rot = (Hq + Hkv) * groups, units = rot + (v ? Hkv * (d / 8) : 0);
    const bool shared_angles = half <= RP_MAX_HALF;
    // (per_wg == 1: a token's units may go to several workgroups, side by side in y)
    const int local = per_wg > 1 ? tid / units : 0;
    const int unit = per_wg > 1 ? tid - local * units : (int)blockIdx.y * RP_THREADS + tid;
    for (int64_t first = (int64_t)blockIdx.x * per_wg; first < n_tokens; first += (int64_t)gridDim.x * per_wg) {
        const int64_t token = first + local;
        const bool live = local < per_wg && token < n_tokens && unit < units, turn = live && unit < rot;
        const int head = unit / groups, grp = unit - head * groups;
        const bool is_q = head < Hq;
        const uint16_t* src = nullptr;
        uint16_t* dst = nullptr;
        uint4 lo = make_uint4(0, 0, 0, 0), hi = lo;
        if (live) {
            const int64_t b = T >= n_tokens ? 0 : (unsigned)token / (unsigned)T;       // (samples: B T < 2^31)
            const int64_t kv_off = b * kv_batch + ((token - b * T) + (rows ? rows[token] : 0)) * Hkv * d;
            if (turn) {
                src = is_q ? q + (token * Hq + head) * d : k + (token * Hkv + (head - Hq)) * d;
                dst = is_q ? q + (token * Hq + head) * d : k_dst + kv_off + (head - Hq) * d;
                src += 8 * grp;
                dst += 8 * grp;
                hi = *reinterpret_cast<const uint4*>(src + half);
            } else {
                const int c = unit - rot;
                src = v + token * Hkv * d + 8 * c;
                dst = v_dst + kv_off + 8 * c;
            }
            lo = *reinterpret_cast<const uint4*>(src);
        }
        auto angle = [&](float pos, int i) {
            float sn, cs;
            sincosf(pos * __builtin_exp2f((float)i * neg_log2_theta_2_over_d), &sn, &cs);
            return make_float2(sn, cs);
        };
        if (shared_angles) {
            for (int i = tid; i < per_wg * half; i += RP_THREADS) {
                const int t = i / half;
                if (first + t < n_tokens) rp_angles[i] = angle((float)positions[first + t], i - t * half);
            }
            __syncthreads();
        }
        if (turn) {
            const uint32_t lw[4] = {lo.x, lo.y, lo.z, lo.w}, hw[4] = {hi.x, hi.y, hi.z, hi.w};
            uint32_t ol[4], oh[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                float rl[2], rh[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 8 * grp + 2 * p + e;
                    const float2 sc = shared_angles ? rp_angles[local * half + i] : angle((float)positions[token], i);
                    const float x = e ? bf16_hi(lw[p]) : bf16_lo(lw[p]);
                    const float y = e ? bf16_hi(hw[p]) : bf16_lo(hw[p]);
                    rl[e] = x * sc.y - y * sc.x;
                    rh[e] = y * sc.y + x * sc.x;
                }
                ol[p] = pack_bf16(rl[0], rl[1]);
                oh[p] = pack_bf16(rh[0], rh[1]);
            }
            *reinterpret_cast<uint4*>(dst) = make_uint4(ol[0], ol[1], ol[2], ol[3]);
            *reinterpret_cast<uint4*>(dst + half) = make_uint4(oh[0], oh[1], oh[2], oh[3]);
        } else if (live) {
            *reinterpret_cast<uint4*>(dst) = lo;
        }
        if (shared_angles) __syncthreads();                // the next tokens' angles replace these
    }
}

int launch_rope_append(uint16_t* q, const uint16_t* k, const uint16_t* v, const int32_t* positions, int64_t n_tokens,
                       int Hq, int Hkv, int d, float theta, uint16_t* k_dst, uint16_t* v_dst, int64_t T,
                       int64_t kv_batch, hipStream_t s, const int32_t* rows) {
    const int64_t units = (int64_t)(Hq + Hkv) * (d / 16) + (v ? (int64_t)Hkv * (d / 8) : 0);
    if (n_tokens == 0 || units == 0) return VITCOP_OK;
    const float c = -2.0f * std::log2(theta) / (float)d;
    const int per_wg = (int)std::max<int64_t>(1, RP_THREADS / units);
    const size_t lds = d / 2 <= RP_MAX_HALF ? (size_t)per_wg * (d / 2) * sizeof(float2) : 0;
    const int64_t wgs = std::min<int64_t>((n_tokens + per_wg - 1) / per_wg, 1 << 20);        // (the kernel walks the rest)
    hipLaunchKernelGGL(rope_kernel, dim3((unsigned)wgs, (unsigned)((units + RP_THREADS - 1) / RP_THREADS)),
                       dim3(RP_THREADS), lds, s, q, k, v, positions, n_tokens, Hq, Hkv, d, c, k_dst, v_dst, T, kv_batch,
                       rows, per_wg);
    return launch_status("rope");
}

int launch_rope(uint16_t* q, uint16_t* k, const int32_t* positions, int64_t n_tokens, int Hq, int Hkv, int d,
                float theta, hipStream_t s) {
    return launch_rope_append(q, k, nullptr, positions, n_tokens, q ? Hq : 0, k ? Hkv : 0, d, theta, k, nullptr,
                              std::max<int64_t>(n_tokens, 1), 0, s);
}

// out = silu(gate) * up, 8 elements per thread
__global__ __launch_bounds__(256) void silu_mul_kernel(const uint16_t* __restrict__ gate,
                                                       const uint16_t* __restrict__ up,
                                                       uint16_t* __restrict__ out, int64_t chunks) {
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= chunks) return;
    const uint4 g = ld_nt16(gate + 8 * c), u = ld_nt16(up + 8 * c);
    auto gated = [](uint32_t gw, uint32_t uw) {
        const float g0 = bf16_lo(gw), g1 = bf16_hi(gw);
        const float s0 = g0 / (1.0f + __expf(-g0)), s1 = g1 / (1.0f + __expf(-g1));
        return pack_bf16(s0 * bf16_lo(uw), s1 * bf16_hi(uw));
    };
    st_nt16(out + 8 * c, make_uint4(gated(g.x, u.x), gated(g.y, u.y), gated(g.z, u.z), gated(g.w, u.w)));
}

int launch_silu_mul(const uint16_t* gate, const uint16_t* up, uint16_t* out, int64_t n_elems, hipStream_t s) {
    const int64_t chunks = n_elems / 8;
    if (chunks == 0) return VITCOP_OK;
    hipLaunchKernelGGL(silu_mul_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, gate, up, out,
                       chunks);
    return launch_status("silu_mul");
}

}  // namespace vitcop
