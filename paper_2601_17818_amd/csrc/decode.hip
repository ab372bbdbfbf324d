// One decoding step over a (compacted) KV cache: o = softmax(scale K q) V for the new token of
// every sample, the per-token cost that pruning the prefill reduces afterwards (Table 5 of
// arXiv 2601.17818 reports it).  HBM-bound: K and V of the cache are read once (once for every 16 query heads of a KV head;
// once more by the wavefronts of decode_group_kernel that meet an infinite value).
//
// decode_partial_kernel: a workgroup takes one KV head, or two or four side by side, and one slice of the keys.  A key row
// (d bf16) is spread over d/8 lanes, 16 bytes each, so a wavefront reads 512/d rows per instruction; every lane keeps its
// 8 query channels, a running maximum, a running sum and 8 output channels (online softmax).  The lane groups, then the
// wavefronts, are merged at the end and one partial (max, sum, unnormalised output) per (sample, head, slice) goes to the
// workspace.
// decode_group_kernel: the same for query heads that share a KV head, whose products go to the matrix cores.
// decode_merge_kernel combines the slices; a single slice is finished on the spot.
#include "vitcop_internal.h"
#include "device_utils.h"

#include <type_traits>

namespace vitcop {

constexpr int DC_THREADS = 256;

struct DecodeGiven {};                       // (in place of DecodeNew: q is given, and the caches hold the new rows)

// The four wavefronts' states of G query heads (sm: maximum and sum, so: unnormalised outputs) combined by threads
// (head, channel): the partial of this slice, or with `out` the output, what decode_merge_kernel makes of one partial.
template <int D, int GMAX, int WAVES = 4>
__device__ __forceinline__ void decode_combine(const float (&sm)[WAVES][GMAX][2], const float (&so)[WAVES][GMAX][D], int G, int b,
                                               int h0, int Hq, int n_splits, int split,
                                               float* __restrict__ part_o, float* __restrict__ part_ml,
                                               uint16_t* __restrict__ out, float* __restrict__ lse) {
    for (int idx = threadIdx.x; idx < G * D; idx += 64 * WAVES) {
        const int g = idx / D, ch = idx - g * D;
        float mn = -INFINITY;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) mn = fmaxf(mn, sm[w][g][0]);
        float lt = 0.f, ot = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float a = mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sm[w][g][0] - mn);
            lt += sm[w][g][1] * a;
            ot += so[w][g][ch] * a;
        }
        if (out != nullptr) {
            const int64_t bh = (int64_t)b * Hq + h0 + g;
            const float r = ot / lt, r1 = __shfl_down(r, 1, 64);         // (a wavefront's lanes share g: D >= 64)
            if ((ch & 1) == 0) *reinterpret_cast<uint32_t*>(out + bh * D + ch) = pack_bf16(r, r1);
            if (lse && ch == 0) lse[bh] = (mn + __builtin_amdgcn_logf(lt)) * 0.6931471805599453f;
            continue;
        }
        const int64_t slot = ((int64_t)b * Hq + h0 + g) * n_splits + split;
        part_o[slot * D + ch] = ot;
        if (ch == 0) {
            part_ml[slot * 2] = mn;
            part_ml[slot * 2 + 1] = lt;
        }
    }
}

// The new token of sample b, where it comes as partial sums: its query heads [hq0, hq0 + n_q) into q_lds, rounded and turned
// as qkv_finish_kernel does, and if `append` says so its rows of KV heads [hk0, hk0 + n_kv) into the caches, from where the
// workgroup reads them like the others (the barrier at the end orders that).  A thread takes two channels that are turned
// together, or two neighbours of v.  Every workgroup of a head puts its q together, a few KB of partial sums and about 1 us
// in front of the stream, which saves the launch that did it for all of them: one layer of a decoding step, us, before and
// now: 4096 / 11008 with 64 samples x 317 keys 158.8, 156.9, x 115 keys 128.5, 124.9, 16 x 317 116.3, 113.0; 3584 / 14336 (28 / 4
// heads) 16 x 115 100.1, 98.5; 2048 / 5632 16 x 300 63.0, 59.8; 1024 / 2816 (16 / 4 heads of 64) 24 x 60 39.4, 35.8.
template <int D, int THREADS>
__device__ __forceinline__ void decode_new_token(const DecodeNew& a, int b, int Hq, int Hkv, int hq0, int n_q, int hk0,
                                                 int n_kv, bool append, int64_t cache_row, uint16_t (*q_lds)[D]) {
    constexpr int HALF = D / 2;
    const float position = (float)a.positions[b];
    const int units_q = n_q * HALF, units_kv = append ? n_kv * HALF : 0;
    const int64_t slice = (int64_t)a.parts.M * a.parts.N;
    for (int u = threadIdx.x; u < units_q + 2 * units_kv; u += THREADS) {
        const bool is_q = u < units_q, is_v = u >= units_q + units_kv;
        const int unit = is_q ? u : (is_v ? u - units_q - units_kv : u - units_q);
        const int head = unit / HALF, i = unit - head * HALF;
        const int c0 = is_v ? 2 * i : i, c1 = is_v ? 2 * i + 1 : i + HALF;
        const int col = (is_q ? Hkv + hq0 : (is_v ? Hkv + Hq + hk0 : hk0)) + head;
        const float* p = a.parts.part + (int64_t)b * a.parts.N + (int64_t)col * D;
        float lo = 0.f, hi = 0.f;
        for (int s0 = 0; s0 < a.parts.slices; s0 += 4) {                 // four slices' loads in flight, added in order
            float x[4], y[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (s0 + t < a.parts.slices) {
                    x[t] = p[(s0 + t) * slice + c0];
                    y[t] = p[(s0 + t) * slice + c1];
                }
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (s0 + t < a.parts.slices) {
                    lo += x[t];
                    hi += y[t];
                }
        }
        uint32_t w = pack_bf16(lo, hi);
        if (!is_v) {
            float sn, cs;
            sincosf(position * __builtin_exp2f((float)i * a.rope_c), &sn, &cs);
            const float l = bf16_lo(w), h = bf16_hi(w);
            w = pack_bf16(l * cs - h * sn, h * cs + l * sn);
        }
        uint16_t* dst = is_q ? q_lds[head] : (is_v ? a.v : a.k) + cache_row + (int64_t)(hk0 + head) * D;
        if (is_v) {
            *reinterpret_cast<uint32_t*>(dst + c0) = w;
        } else {
            dst[c0] = (uint16_t)w;
            dst[c1] = (uint16_t)(w >> 16);
        }
    }
    __syncthreads();
}

// One query head per KV head (G = 1), or two where group_on_vectors says so.  HBM-bound.  HEADS neighbouring heads' rows of
// a key lie side by side in the cache, and a wavefront reads them together: pieces of 512 bytes and more instead of 256 at a
// stride of Hkv * 2 D bytes (64 samples x 32 heads x 318 keys 59.6 -> 54.0 us, 5.6 -> 6.2 TB/s; x 118 keys 24.0 -> 22.1; x 640
// keys 115.8 -> 102.2, 6.6 TB/s).  Four wavefronts per head as before, so the keys of each wavefront, and the loads in flight,
// are the same number.
// AHEAD: the next rows of K and V are requested before the current ones are used.  Pays for slices of a few hundred
// keys (one head at a time: 64 samples x 32 heads x 318 keys 61.7 -> 57.6 us, 5.4 -> 5.8 TB/s; x 116 keys 26.4 -> 23.9); not
// for long ones (32 x 4096 keys 305 -> 321 us), nor with two query heads, which have work to do meanwhile.
constexpr int DC_AHEAD_MAX_KEYS = 1024;
template <int D, bool AHEAD, int HEADS, int G, typename New>
__global__ __launch_bounds__(DC_THREADS * HEADS) void decode_partial_kernel(
    const uint16_t* __restrict__ q, const uint16_t* k, const uint16_t* v,
    float* __restrict__ part_o, float* __restrict__ part_ml, int N, int H, float scale_log2e, int keys_per_split,
    int n_splits, int64_t kv_batch, const int32_t* __restrict__ n_cached_samples, uint16_t* __restrict__ out,
    float* __restrict__ lse, New fresh) {
    constexpr bool FRESH = std::is_same<New, DecodeNew>::value;
    constexpr int LPK = D / 8;                       // lanes per key row of a head
    constexpr int KPW = 64 / (LPK * HEADS);          // keys per wavefront instruction
    constexpr int WAVES = 4 * HEADS;
    const int split = blockIdx.x, h0 = blockIdx.y * HEADS, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = lane % LPK, kq = lane / (LPK * HEADS), hs = lane / LPK % HEADS, h = h0 + hs;

    // caches of different lengths: sample b attends over its n_cached_samples[b] rows and the appended one;
    // slices past them see no live key and hand on an empty partial (max -inf, sum 0)
    const int n_keys = n_cached_samples ? min(max(n_cached_samples[b], 0) + 1, N) : N;
    const int key_begin = split * keys_per_split, key_end = min(n_keys, key_begin + keys_per_split);
    const int64_t row = (int64_t)H * D;
    const uint16_t* kb = k + b * kv_batch + h * D + 8 * c;       // kv_batch: elements between two samples' caches
    const uint16_t* vb = v + b * kv_batch + h * D + 8 * c;
    const int key_first = key_begin + wv * KPW;
    uint4 k_next = make_uint4(0, 0, 0, 0), v_next = k_next;
    auto first_rows = [&]() __attribute__((always_inline)) {
        const int kc = min(key_first + kq, key_end - 1);
        k_next = ld_nt16(kb + kc * row);
        v_next = ld_nt16(vb + kc * row);
    };
    // (the first rows are on their way while the new token is put together, unless the last one, its own, is among them)
    const bool early = FRESH && AHEAD && key_first < key_end && key_first + KPW < n_keys;
    const uint16_t* q_row = nullptr;
    if constexpr (FRESH) {
        __shared__ alignas(16) uint16_t q_new[HEADS * G][D];
        if (early) first_rows();
        decode_new_token<D, DC_THREADS * HEADS>(fresh, b, H * G, H, h0 * G, HEADS * G, h0, HEADS,
                                                key_begin < n_keys && key_end == n_keys,
                                                b * kv_batch + (n_keys - 1) * row, q_new);
        q_row = &q_new[hs * G][8 * c];
    } else {
        q_row = q + ((int64_t)b * H + h) * G * D + 8 * c;
    }
    float qv[G][8], m[G], l[G], acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const uint4 u = *reinterpret_cast<const uint4*>(q_row + g * D);
        qv[g][0] = bf16_lo(u.x); qv[g][1] = bf16_hi(u.x); qv[g][2] = bf16_lo(u.y); qv[g][3] = bf16_hi(u.y);
        qv[g][4] = bf16_lo(u.z); qv[g][5] = bf16_hi(u.z); qv[g][6] = bf16_lo(u.w); qv[g][7] = bf16_hi(u.w);
        m[g] = -INFINITY;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[g][e] = 0.f;
    }
    if (AHEAD && !early && key_first < key_end) first_rows();
    for (int key0 = key_first; key0 < key_end; key0 += WAVES * KPW) {     // (empty if key_end <= key_begin)
        const int key = key0 + kq;
        const bool live = key < key_end;
        uint4 ku, vu;
        if constexpr (AHEAD) {
            ku = k_next;
            vu = v_next;
            if (key0 + WAVES * KPW < key_end) {                           // (uniform in the wavefront)
                const int kc = min(key + WAVES * KPW, key_end - 1);
                k_next = ld_nt16(kb + kc * row);
                v_next = ld_nt16(vb + kc * row);
            }
        } else {
            const int kc = min(key, key_end - 1);
            ku = ld_nt16(kb + kc * row);
            vu = ld_nt16(vb + kc * row);
        }
        // a slot past the end holds a copy of the last row: the zero probability of an infinite value would be NaN
        if (KPW > 1 && !live) vu = make_uint4(0, 0, 0, 0);
        const float kf[8] = {bf16_lo(ku.x), bf16_hi(ku.x), bf16_lo(ku.y), bf16_hi(ku.y),
                             bf16_lo(ku.z), bf16_hi(ku.z), bf16_lo(ku.w), bf16_hi(ku.w)};
        const float vf[8] = {bf16_lo(vu.x), bf16_hi(vu.x), bf16_lo(vu.y), bf16_hi(vu.y),
                             bf16_lo(vu.z), bf16_hi(vu.z), bf16_lo(vu.w), bf16_hi(vu.w)};
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) s = fmaf(qv[g][e], kf[e], s);
#pragma unroll
            for (int o = LPK / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);      // over the lanes of this key
            s = live ? s * scale_log2e : -INFINITY;
            const float m_new = fmaxf(m[g], s);
            // m_new is -inf only while nothing live has been seen: then alpha and p must be 0, not NaN
            const float alpha = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[g] - m_new);
            const float p = m_new == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s - m_new);
            m[g] = m_new;
            l[g] = fmaf(l[g], alpha, p);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] = fmaf(acc[g][e], alpha, p * vf[e]);
        }
    }
    // merge the KPW key sub-groups of the wavefront (lanes with the same c), then the wavefronts
    __shared__ float sm[WAVES][HEADS * G][2];
    __shared__ float so[WAVES][HEADS * G][D];
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int o = LPK * HEADS; o < 64; o <<= 1) {
            const float mo = __shfl_xor(m[g], o, 64), lo = __shfl_xor(l[g], o, 64);
            const float mn = fmaxf(m[g], mo);
            const float a0 = mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[g] - mn);
            const float a1 = mn == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mo - mn);
            l[g] = l[g] * a0 + lo * a1;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[g][e] = acc[g][e] * a0 + __shfl_xor(acc[g][e], o, 64) * a1;
            m[g] = mn;
        }
        if (kq == 0) {
            if (c == 0) {
                sm[wv][hs * G + g][0] = m[g];
                sm[wv][hs * G + g][1] = l[g];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) so[wv][hs * G + g][8 * c + e] = acc[g][e];
        }
    }
    __syncthreads();
    decode_combine<D, HEADS * G, WAVES>(sm, so, HEADS * G, b, h0 * G, H * G, n_splits, split, part_o, part_ml, out, lse);
}

// Query heads that share a KV head (2 to 16 of them a pass).  On the vector pipe every key costs each of them 16 FMAs a
// lane, a reduction over lanes and an exponential: 64 samples x 318 keys x 28 / 4 heads x 128 took 45 us for 42 MB (now
// 12.5), 32 x 4096 keys 121 (51), 64 x 400 x 16 / 4 x 64 20.8 (8.7), 64 x 318 x 32 / 16 37.6 (33.9); where that is still the
// faster way: group_on_vectors.  Here a wavefront
// takes 32 keys at a time: scores S^T = K Q^T (16x16x32: a lane holds 4 keys of one head), the softmax with the lane's
// head as its only query, and O^T += V^T P^T, V transposed on the way out of LDS (ds_read_b64_tr_b16).  The key of
// element 4 t + r of a lane's 8 in the second product is 16 t + 4 (lane / 16) + r, which is where the scores are.  The
// probabilities stay 32-bit: each is the sum of three bf16 (24 bits), one product for each.
// Registers for three workgroups on a CU (d = 64: four): many pairs of a few keys are a chain of latencies each, which
// only other workgroups fill (us with two and with three: 250 samples x 40 keys x 32 / 16 x 128 35.2, 30.2; x 100 x 28 / 4
// 16.2, 14.9; where the keys are many it is the loads that count, 64 x 2000 x 28 / 4 47.6, 47.9).
constexpr int DG_MAX_G = 16, DG_KEYS = 32;
template <int D, typename New>
__global__ __launch_bounds__(DC_THREADS, D == 128 ? 3 : 4) void decode_group_kernel(
    const uint16_t* __restrict__ q, const uint16_t* k, const uint16_t* v,
    float* __restrict__ part_o, float* __restrict__ part_ml, int N, int Hq, int Hkv, int g0, int G,
    float scale_log2e, int keys_per_split, int n_splits, int64_t kv_batch,
    const int32_t* __restrict__ n_cached_samples, uint16_t* __restrict__ out, float* __restrict__ lse, New fresh) {
    constexpr bool FRESH = std::is_same<New, DecodeNew>::value;
    constexpr int STEPS = D / 32, BLOCKS = D / 16;
    constexpr int VROW = 2 * D + 32;                         // bytes of a V row in LDS: the pad keeps eight rows apart
    constexpr int LPR = D / 8, RPL = 64 / LPR, VL = DG_KEYS / RPL;         // lanes a row, rows a load, loads a tile of V
    static_assert(DG_KEYS * VROW >= DG_MAX_G * D * 4, "the outputs take V's place at the end");
    __shared__ __attribute__((aligned(16))) char vt[4][DG_KEYS * VROW];
    __shared__ float sm[4][DG_MAX_G][2];
    float (&so)[4][DG_MAX_G][D] = *reinterpret_cast<float (*)[4][DG_MAX_G][D]>(&vt[0][0]);
    const int split = blockIdx.x, hk = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, l16 = lane & 15, g4 = lane >> 4;
    const int group = Hq / Hkv, h0 = hk * group + g0;        // first query head of this pass
    const int n_keys = n_cached_samples ? min(max(n_cached_samples[b], 0) + 1, N) : N;
    const int key_begin = split * keys_per_split, key_end = min(n_keys, key_begin + keys_per_split);
    const int64_t row = (int64_t)Hkv * D;
    const uint16_t* kb = k + b * kv_batch + hk * D;
    const uint16_t* vb = v + b * kv_batch + hk * D;

    f32x4 o[BLOCKS];
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;                            // of head l16 (m over all its keys, l over this lane's)

    // Rows past the end: of K the last one, masked below; of V zeros, for which the descriptor ends with the last row (a
    // copy would not do: the zero probability of an infinite value is NaN).  A sample's cache is below 4 GiB.
    const unsigned row_b = (unsigned)row * 2;
    const auto v_desc = __builtin_amdgcn_make_buffer_rsrc((void*)vb, 0, (key_end - 1) * row_b + 2 * D, 0x00020000);
    u32x4 kr[2][STEPS], vr[VL];
    auto load = [&](int key0) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint16_t* p = kb + min(key0 + 16 * t + l16, key_end - 1) * row + 8 * g4;
#pragma unroll
            for (int c = 0; c < STEPS; ++c) kr[t][c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + 32 * c));
        }
#pragma unroll
        for (int i = 0; i < VL; ++i)
            vr[i] = __builtin_amdgcn_raw_buffer_load_b128(
                v_desc, min(key0 + RPL * i + lane / LPR, key_end) * row_b + 16 * (lane % LPR), 0, 2 /* non-temporal */);
    };
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    char* const mine = vt[wv];
    const unsigned tr = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)mine +
                        (4 * g4 + ((lane >> 2) & 3)) * VROW + (lane & 3) * 8;
    const int first = key_begin + wv * DG_KEYS;
    const bool early = FRESH && first + DG_KEYS < n_keys && first < key_end;      // (as in decode_partial_kernel)
    if (early) load(first);
    bf16x8 qf[STEPS];                                        // Q^T: 8 channels of head l16 a step (heads past G: head G - 1)
    if constexpr (FRESH) {
        __shared__ alignas(16) uint16_t q_new[DG_MAX_G][D];
        decode_new_token<D, DC_THREADS>(fresh, b, Hq, Hkv, h0, G, hk, 1, g0 == 0 && key_begin < n_keys && key_end == n_keys,
                                        b * kv_batch + (n_keys - 1) * row, q_new);
#pragma unroll
        for (int c = 0; c < STEPS; ++c) qf[c] = *reinterpret_cast<const bf16x8*>(&q_new[min(l16, G - 1)][32 * c + 8 * g4]);
    } else {
#pragma unroll
        for (int c = 0; c < STEPS; ++c)
            qf[c] = *reinterpret_cast<const bf16x8*>(q + ((int64_t)b * Hq + h0 + min(l16, G - 1)) * D + 32 * c + 8 * g4);
    }
    auto attend = [&](auto parts_c) __attribute__((always_inline)) {     // PARTS: bf16 summands of a probability
        constexpr int PARTS = decltype(parts_c)::value;
        constexpr bool AHEAD = PARTS > 1;                    // (the registers of the second pass hold the first's outputs)
        if (AHEAD && !early && first < key_end) load(first);
        for (int key0 = first; key0 < key_end; key0 += 4 * DG_KEYS) {
            if (!AHEAD) load(key0);
            f32x4 s[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < STEPS; ++c)
                    s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[t][c]), qf[c], s[t], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < VL; ++i)
                *reinterpret_cast<u32x4*>(mine + (RPL * i + lane / LPR) * VROW + lane % LPR * 16) = vr[i];
            if (AHEAD && key0 + 4 * DG_KEYS < key_end) load(key0 + 4 * DG_KEYS);      // (uniform) in flight from here on
            float p[8], top = -INFINITY;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int key = key0 + 16 * (e >> 2) + 4 * g4 + (e & 3);
                p[e] = key < key_end ? s[e >> 2][e & 3] * scale_log2e : -INFINITY;
                top = fmaxf(top, p[e]);
            }
            top = fmaxf(top, __shfl_xor(top, 16, 64));
            top = fmaxf(top, __shfl_xor(top, 32, 64));
            const float m_new = fmaxf(m, top);
            const float base = m_new == -INFINITY ? 0.f : m_new;         // (nothing but -inf so far: 0, not NaN)
            const float alpha = __builtin_amdgcn_exp2f(m - base);
            m = m_new;
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                p[e] = __builtin_amdgcn_exp2f(p[e] - base);
                sum += p[e];
            }
            l = fmaf(l, alpha, sum);
            u32x4 part[PARTS];                               // the rest of the rest last
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float a = p[2 * e], c = p[2 * e + 1];
#pragma unroll
                for (int n = 0; n < PARTS; ++n) {
                    const uint32_t w = pack_bf16(a, c);
                    part[n][e] = w;
                    a -= bf16_lo(w);
                    c -= bf16_hi(w);
                }
            }
            if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
                for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[i][r] *= alpha;
            }
            __builtin_amdgcn_wave_barrier();                     // (one wavefront's LDS accesses stay in order)
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i) {
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4*)(uintptr_t)(tr + i * 32));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4*)(uintptr_t)(tr + i * 32 + 16 * VROW));
                const bf16x8 vf = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
                for (int n = 0; n < PARTS; ++n)
                    o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, part[n]), o[i], 0, 0, 0);
            }
            __builtin_amdgcn_wave_barrier();                     // the next tile's rows replace these
        }
    };
    attend(std::integral_constant<int, 3>{});
    // An infinite value of V times a zero among the later parts of its probability is no number: such outputs (alone)
    // are summed again with the first parts only, of which one is zero only where the probability itself is.
    bool nan = false;
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) nan |= o[i][r] != o[i][r];
    if (__builtin_amdgcn_ballot_w64(nan) != 0) {
        f32x4 sums[BLOCKS];
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i) {
            sums[i] = o[i];
            o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        m = -INFINITY;
        l = 0.f;
        attend(std::integral_constant<int, 1>{});
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (sums[i][r] == sums[i][r]) o[i][r] = sums[i][r];
    }
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    __syncthreads();                                         // all are done with V
    if (g4 == 0) {
        sm[wv][l16][0] = m;
        sm[wv][l16][1] = l;
    }
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i) *reinterpret_cast<f32x4*>(&so[wv][l16][16 * i + 4 * g4]) = o[i];
    __syncthreads();
    decode_combine<D, DG_MAX_G>(sm, so, G, b, h0, Hq, n_splits, split, part_o, part_ml, out, lse);
}

template <int D>
__global__ __launch_bounds__(D) void decode_merge_kernel(const float* __restrict__ part_o,
                                                         const float* __restrict__ part_ml, int n_splits,
                                                         uint16_t* __restrict__ out, float* __restrict__ lse) {
    const int64_t bh = blockIdx.x;
    const int ch = threadIdx.x;
    float mn = -INFINITY;
    for (int s = 0; s < n_splits; ++s) mn = fmaxf(mn, part_ml[(bh * n_splits + s) * 2]);
    float lt = 0.f, ot = 0.f;
    for (int s = 0; s < n_splits; ++s) {
        const float ms = part_ml[(bh * n_splits + s) * 2];
        const float a = ms == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms - mn);
        lt += part_ml[(bh * n_splits + s) * 2 + 1] * a;
        ot += part_o[(bh * n_splits + s) * D + ch] * a;
    }
    const float r = ot / lt;
    // neighbouring channels pair up into one 32-bit store
    const float r1 = __shfl_down(r, 1, 64);
    if ((ch & 1) == 0) *reinterpret_cast<uint32_t*>(out + bh * D + ch) = pack_bf16(r, r1);
    if (lse && ch == 0) lse[bh] = (mn + __builtin_amdgcn_logf(lt)) * 0.6931471805599453f;
}

int decode_splits(int B, int N, int Hkv) {
    // about four workgroups per CU, slices of at least 64 keys
    const long wgs = (long)B * Hkv;
    long s = (1024 + wgs - 1) / wgs;
    const long max_s = (N + 63) / 64;
    if (s > max_s) s = max_s;
    if (s < 1) s = 1;
    return (int)s;
}

// Slices for decode_group_kernel, never more than the above, which sizes the scratch: its wavefronts keep 16 KB each in
// flight, so it needs fewer, of at least 128 keys (32 a wavefront), and with one there is no merge.
constexpr int DG_WGS = 256;
static int group_splits(int B, int N, int Hkv) {
    const long wgs = (long)B * Hkv;
    return (int)std::max(1L, std::min((DG_WGS + wgs - 1) / wgs, (N + 127L) / 128));
}

// Two query heads to a KV head (`pairs`: of a sample and a KV head) go to decode_partial_kernel where a workgroup's tile of
// 128 keys is mostly empty, the more so the more pairs wait for their turn, and where the pairs are so many that the bytes
// alone count, which its small workgroups draw faster.  On the matrix cores and on this kernel, us, of 128 channels: 16 pairs
// x 16 keys 4.5, 3.9, x 48 4.8, 5.2; 512 x 32 7.0, 6.6, x 48 7.6, 7.9; 2000 x 16 16.3, 9.5, x 64 20.7, 19.2, x 100 24.0, 27.6;
// 8000 x 16 55, 27, x 317 238, 217; 4000 x 100 42, 44, x 640 236, 230.  Of 64 channels: 4000 x 16 16.3, 15.5, x 64 21.1, 21.8,
// x 100 25.4, 29.2, x 317 71, 67; 2048 x 317 38.7, 42.4; 8000 x 640 279, 234.  Three and four query heads were faster there
// up to 16 keys alone (8000 pairs x 8 keys x 4 heads 58, 52; x 32 58, 69), more of them at no size.
static bool group_on_vectors(long pairs, int N, int group, int d) {
    if (group != 2) return false;
    if (pairs > 12 * 256) return d == 128 || N <= 16 || N > 128;
    return d == 128 && N <= std::max(16L, std::min(64L, pairs / 16));
}

// Heads that decode_partial_kernel reads side by side: what the fullest CU gets to do, `pairs` (sample, head, slice)
// dealt out `heads` at a time, times the time of one against that of reading 256 bytes a row.  Four leave a CU with one
// workgroup, and nothing beside its start and end, unless there are more than 256 such.  Measured, us in one, two and four:
// 64 samples x 32 heads x 353 keys 64.7, 58.4, 58.5; 44 x 32 x 353 43.9, 39.6, 47.1; 25 x 40 x 700 68.7, 65.4, 61.5;
// 26 x 40 x 700 66.1, 71.5, 82.6; 32 x 32 x 1000 80.4, 77.3, 81.9; 128 x 16 (of 64 channels) x 200 21.7, 20.3, 19.2.
static int heads_side_by_side(long pairs, int heads) {
    int best = 1;
    float least = (float)((pairs + 255) / 256);
    for (int n : {2, 4}) {
        if (heads % n != 0 || (n == 4 && pairs <= 4 * 256)) continue;
        const float load = (float)((pairs + 256 * n - 1) / (256 * n) * n) * (n == 2 ? 0.9f : 0.88f);
        if (load <= least) {
            least = load;
            best = n;
        }
    }
    return best;
}

size_t decode_workspace_bytes(int B, int N, int Hq, int Hkv, int d) {
    const size_t s = decode_splits(B, N, Hkv);
    return up256((size_t)B * Hq * s * d * 4) + up256((size_t)B * Hq * s * 2 * 4);
}

template <int D, typename New>
static int launch_decode_d(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out, float* lse,
                           int B, int N, int Hq, int Hkv, float scale, void* ws, hipStream_t s, int64_t kv_batch,
                           DecodeParts* hand_over, const int32_t* ncs, const New& fresh) {
    const bool on_vectors = Hq > Hkv && group_on_vectors((long)B * Hkv, N, Hq / Hkv, D), grouped = Hq > Hkv && !on_vectors;
    const int ns = grouped ? group_splits(B, N, Hkv) : decode_splits(B, N, Hkv);
    const int kps = ((N + ns - 1) / ns + 63) / 64 * 64;
    float* po = static_cast<float*>(ws);
    float* pml = reinterpret_cast<float*>(static_cast<char*>(ws) + up256((size_t)B * Hq * ns * D * 4));
    const float sl2 = scale * 1.4426950408889634f;
    const int group = Hq / Hkv;
    dim3 grid(ns, Hkv, B);
    // one slice (few keys, or as many (sample, KV head) pairs as four workgroups per CU, of grouped heads as one): the
    // outputs are written right away and the merge's launch is saved (64 samples x 32 heads: 4.9 us a layer)
    uint16_t* o1 = ns == 1 ? out : nullptr;
    if (grouped) {
        for (int g0 = 0; g0 < group; g0 += DG_MAX_G) {
            hipLaunchKernelGGL((decode_group_kernel<D, New>), grid, dim3(DC_THREADS), 0, s, q, k, v, po, pml, N, Hq, Hkv, g0,
                               std::min(DG_MAX_G, group - g0), sl2, kps, ns, kv_batch, ncs, o1, lse, fresh);
            const int rc = launch_status("decode_group");
            if (rc) return rc;
        }
    } else {
        const bool ahead = kps <= DC_AHEAD_MAX_KEYS;
        const int heads = on_vectors ? 1 : heads_side_by_side((long)B * Hkv * ns, Hkv);
        auto* kernel = ahead ? decode_partial_kernel<D, true, 1, 1, New> : decode_partial_kernel<D, false, 1, 1, New>;
        if (heads == 2) kernel = ahead ? decode_partial_kernel<D, true, 2, 1, New> : decode_partial_kernel<D, false, 2, 1, New>;
        if (heads == 4) kernel = ahead ? decode_partial_kernel<D, true, 4, 1, New> : decode_partial_kernel<D, false, 4, 1, New>;
        if (on_vectors) kernel = decode_partial_kernel<D, false, 1, 2, New>;
        grid.y = Hkv / heads;
        hipLaunchKernelGGL(kernel, grid, dim3(DC_THREADS * heads), 0, s, q, k, v, po, pml, N, Hkv, sl2, kps, ns, kv_batch, ncs,
                           o1, lse, fresh);
        const int rc = launch_status("decode_partial");
        if (rc) return rc;
    }
    if (ns == 1) {
        if (hand_over != nullptr) *hand_over = DecodeParts{nullptr, nullptr, 0};
        return VITCOP_OK;
    }
    if (hand_over != nullptr && ns <= DECODE_PARTS_MAX_SPLITS) {       // the caller's next kernel combines the slices
        *hand_over = DecodeParts{po, pml, ns};
        return VITCOP_OK;
    }
    if (hand_over != nullptr) *hand_over = DecodeParts{nullptr, nullptr, 0};
    hipLaunchKernelGGL((decode_merge_kernel<D>), dim3((unsigned)(B * Hq)), dim3(D), 0, s, po, pml, ns, out, lse);
    return launch_status("decode_merge");
}

int launch_decode_attn(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out, float* lse, int B,
                       int N, int Hq, int Hkv, int d, float scale, void* ws, hipStream_t s, int64_t kv_batch,
                       DecodeParts* hand_over, const int32_t* n_cached_samples, const DecodeNew* fresh) {
    if (kv_batch == 0) kv_batch = (int64_t)N * Hkv * d;         // dense caches
    auto go = [&](auto launch, const auto& token) {
        return launch(q, k, v, out, lse, B, N, Hq, Hkv, scale, ws, s, kv_batch, hand_over, n_cached_samples, token);
    };
    if (fresh != nullptr && fresh->parts.part != nullptr)
        return d == 64 ? go(launch_decode_d<64, DecodeNew>, *fresh) : go(launch_decode_d<128, DecodeNew>, *fresh);
    return d == 64 ? go(launch_decode_d<64, DecodeGiven>, DecodeGiven{}) : go(launch_decode_d<128, DecodeGiven>, DecodeGiven{});
}

}  // namespace vitcop
