// Linear projection y = x W^T on the bf16 matrix cores, with the K-vector
// norm of Eq. 4 (Sec. 3.2.2) produced in the epilogue: per row, the sum of
// squares of the rounded outputs of each group of 128 columns is written as
// one deterministic partial, so the selection pass never re-reads K.
//
// x [M,K] and W [N,K] are both contiguous along the contraction index, so the
// two MFMA operands are fetched the same way: a lane reads 8 consecutive
// k-values of one row.  The product is formed transposed (W tile as the A
// operand, x tile as the B operand): a lane then owns one output row m and
// 4-element runs of consecutive columns n, which gives 8-byte stores and
// in-lane row sums for the norm epilogue.
//
// Pipeline: k-steps of 64 held in a ring of LDS slabs that are filled by direct global -> LDS
// buffer loads (no register staging); one barrier per k-step; the instruction stream of a step is
// laid out slot by slot, one MFMA per slot, with the fragment reads and loads of the steps to come
// behind them.  Workgroups are renumbered so that each XCD (own L2) works on a compact patch of
// output tiles.
#include <algorithm>
#include <atomic>
#include <type_traits>
#include <utility>
#include "vitcop_internal.h"
#include "device_utils.h"

namespace vitcop {

constexpr int GM_THREADS = 256;
constexpr int GM_PART = 128;         // columns per sum-of-squares partial
[[maybe_unused]] constexpr int GM_XCDS = 8;

// LDS: the slab ring, reused by the epilogue as one staging region per wavefront of
// (BM / WAVES_M) rows of (BN / WAVES_N) bf16 + 16 bytes of padding.
template <int BM, int BN, int WAVES_M, int WAVES_N, int NS>
constexpr size_t gemm_lds_bytes() {
    constexpr size_t ring = (size_t)NS * (BM + BN) * 128;
    constexpr size_t stage = (size_t)4 * (BM / WAVES_M) * ((BN / WAVES_N) * 2 + 16);
    return ring > stage ? ring : stage;
}

// calls f with the compile-time indices 0 .. N-1 (a `#pragma unroll` of this many slots is not honoured)
template <int... I, typename F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// A slab row holds 64 bf16 (128 bytes: whole lines, unpadded because direct loads write 1 KiB runs).
// 16-byte chunk c of row r lives at chunk position c ^ gm_swz(r), which makes the MFMA fragment
// reads (16 consecutive rows, same chunk) bank-conflict free: LDS serves a 16-byte read 16 lanes at a
// time, so 16 consecutive rows must fall on the 16 different 16-byte units of a 256-byte bank row.  The
// unit is 8*(r & 1) + position, so the position must differ among the eight rows of equal parity.
__device__ __forceinline__ int gm_swz(int row) { return (row >> 1) & 7; }

// y = x W^T (+ residual).  With w2 != nullptr the columns [n_split, N) come from a second weight
// matrix and go to a second output (two projections of the same input in one launch).
// EPI selects the epilogue: GM_EPI_BF16 the projection described above; GM_EPI_DIST writes,
// in fp32, the Euclidean distance between row m of x and row n of w from their inner product
// and the two squared row norms: dist[m,n] = sqrt(max(0, xsq[m] + wsq[n] - 2 <x_m, w_n>)).
// GM_EPI_PART is split-K: blockIdx.y = split, which multiplies its share of the k-steps and writes the
// raw fp32 accumulators to dist[split][m][n] (row stride dist_stride, slices dist_batch apart) for a
// reduction kernel to add up.
// GM_EPI_GATED is the MLP's first half in one launch: a tile's first BN/2 columns are rows of w (gate), its
// last BN/2 the same rows of w2 (up); N counts the columns of each; the epilogue rounds both to bf16 as the
// two separate projections would, and stores y[m,n] = silu(gate[m,n]) * up[m,n] (WAVES_N == 2: the gate
// columns of a tile belong to the wavefronts with wn = 0, the up columns to wn = 1).
constexpr int GM_EPI_BF16 = 0, GM_EPI_DIST = 1, GM_EPI_PART = 2, GM_EPI_GATED = 3;

// What bounds the big tiles is power: with the matrix cores 87 % busy the clock falls to 1.7 GHz on random
// operands.  To get there the loop must keep issuing MFMAs.  16x16x32 instructions (half the accumulator
// traffic per FLOP of 32x32x16) in an order fixed by sched_barrier, each pinned to accumulation registers by an
// asm constraint (left to itself the allocator moves 60 % as many registers as there are MFMAs); k-steps of 64
// (every direct load moves 8 whole lines), for the 256-column tiles in two slabs: one barrier per step, loads
// one per four MFMAs right behind it so that a CU's load path (64 bytes per clock) is never asked for more than
// it moves and no wavefront is stuck on issuing one.  Against 32x32x16 with four slabs of 32 and compiler
// scheduling hints (GPU time, random operands, same box): 11776x4096x4096 354 -> 298 us (1116 -> 1326 TFLOP/s),
// 8192x8192x8192 921 -> 750 us (1194 -> 1467), 1536x8192x4096 107 -> 93 us, 2536x4096x11008 229 -> 194 us.
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int NS>
__global__ __launch_bounds__(GM_THREADS) void gemm_kernel(
    const uint16_t* __restrict__ x, int64_t x_stride, const uint16_t* __restrict__ w,
    uint16_t* __restrict__ y, int64_t y_stride, const uint16_t* __restrict__ res,
    int64_t res_stride, int M, int N, int K, float* __restrict__ sumsq_parts, int tiles_m,
    int tiles_n, int group_m, const uint16_t* __restrict__ w2, uint16_t* __restrict__ y2,
    int n_split, int64_t w_stride, const float* __restrict__ xsq, const float* __restrict__ wsq,
    float* __restrict__ dist, int64_t dist_stride, int64_t x_batch, int64_t sq_batch,
    int64_t dist_batch) {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(WAVES_M * WAVES_N == 4, "four wavefronts");
    constexpr int TM = BM / WAVES_M, TN = BN / WAVES_N;
    constexpr int MI = TM / 16, NI = TN / 16;
    constexpr int ROWB = 128;                            // bytes per slab row
    constexpr int SLAB = (BM + BN) * ROWB;               // bytes per slab
    constexpr int NL = SLAB / 4096;                      // direct loads per wavefront per slab
    constexpr int NM = MI * NI, NR = MI + NI;            // MFMAs and fragment reads per 32-wide slice of k
    static_assert(BM % 32 == 0 && BN % 32 == 0, "a load of the four wavefronts covers 32 rows of one operand");

    extern __shared__ __attribute__((aligned(1024))) char gemm_lds[];
    if constexpr (EPI == GM_EPI_PART) dist += blockIdx.y * dist_batch;
    if constexpr (EPI == GM_EPI_DIST) {      // blockIdx.y = image: x and w are the same feature matrix
        x += blockIdx.y * x_batch;
        w += blockIdx.y * x_batch;
        xsq += blockIdx.y * sq_batch;
        wsq += blockIdx.y * sq_batch;
        dist += blockIdx.y * dist_batch;
    }

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);      // wavefront index, kept scalar
    const int l16 = lane & 15, g4 = lane >> 4;
    const int wm = wv % WAVES_M, wn = wv / WAVES_M;

    // Workgroup -> tile.  Consecutive workgroup ids go to different XCDs, so id % 8 picks the
    // XCD and id / 8 the slot inside it; each XCD walks a contiguous range of a grouped
    // ordering (group_m tile rows by all tile columns, column-major inside the group).
    int tile_m, tile_n;
    {
        const int nt = tiles_m * tiles_n;
        const int pid = blockIdx.x;
        const int per = (nt + GM_XCDS - 1) / GM_XCDS;
        int lin = (pid % GM_XCDS) * per + pid / GM_XCDS;
        if (nt % GM_XCDS != 0) lin = pid;             // ragged: plain order
        const int width = group_m * tiles_n;
        const int grp = lin / width;
        const int first = grp * group_m;
        const int gsz = min(tiles_m - first, group_m);
        const int in = lin - grp * width;
        tile_m = first + in % gsz;
        tile_n = in / gsz;
    }
    const int m0 = tile_m * BM;
    int n0 = tile_n * (EPI == GM_EPI_GATED ? BN / 2 : BN);
    if constexpr (EPI == GM_EPI_GATED) {
        static_assert(EPI != GM_EPI_GATED || WAVES_N == 2, "gate and up halves go to the two wavefront columns");
    } else if (w2 != nullptr && n0 >= n_split) {         // second projection (uniform per workgroup)
        w = w2;
        y = y2;
        n0 -= n_split;
        N -= n_split;
        if constexpr (EPI == GM_EPI_PART) dist += n_split;       // the partials keep the launch's column index
    } else if (w2 != nullptr) {
        N = n_split;
    }

    f32x4 acc[NI][MI];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Direct global -> LDS loads.  Load q of wavefront wv fills the 1 KiB of slab rows [32 q + 8 wv, + 8): lane L
    // lands at row L / 8, chunk position L % 8, so it must fetch the chunk that the swizzle assigns to that
    // position.  Rows [0,BM) are x, then W (gated: BN/2 gate rows, then the same rows of up).  One descriptor
    // per operand covers this tile's rows: rows past the end of the matrix, and k-steps past the end of the
    // range (whose scalar offset is the descriptor's size), are out of range: they move nothing and read as zeros.
    const int rows_x = min(M - m0, BM), rows_w = min(N - n0, EPI == GM_EPI_GATED ? BN / 2 : BN);
    const unsigned rec_x = 2u * ((unsigned)(rows_x - 1) * (unsigned)x_stride + (unsigned)K);
    const unsigned rec_w = 2u * ((unsigned)(rows_w - 1) * (unsigned)w_stride + (unsigned)K);
    auto descriptor = [](const uint16_t* base, unsigned bytes) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);     // raw buffer, 32-bit data format
    };
    const auto desc_x = descriptor(x + (int64_t)m0 * x_stride, rec_x);
    const auto desc_w = descriptor(w + (int64_t)n0 * w_stride, rec_w);
    const auto desc_u = descriptor((EPI == GM_EPI_GATED ? w2 : w) + (int64_t)n0 * w_stride, rec_w);
    unsigned goff[NL];               // byte offset of this lane's chunk from its descriptor's base at k = 0
    const unsigned chunk = (unsigned)((lane % 8) ^ gm_swz(8 * wv + lane / 8)) * 16;     // (the same for every q)
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int row = 32 * q + 8 * wv + lane / 8;                             // slab row
        const int wrow = EPI == GM_EPI_GATED && row - BM >= BN / 2 ? row - BM - BN / 2 : row - BM;
        goff[q] = (row < BM ? 2u * (unsigned)row * (unsigned)x_stride : 2u * (unsigned)wrow * (unsigned)w_stride) + chunk;
    }
    auto issue_load = [&](auto q_c, int slab_off, unsigned kx, unsigned kw, unsigned past) __attribute__((always_inline)) {
        constexpr int q = decltype(q_c)::value;
        const unsigned off = goff[q] | past;
        auto dst = (__attribute__((address_space(3))) void*)(gemm_lds + slab_off + (4 * q + wv) * 1024);
        if constexpr (32 * q < BM) __builtin_amdgcn_raw_ptr_buffer_load_lds(desc_x, dst, 16, off, kx, 0, 0);
        else if constexpr (EPI == GM_EPI_GATED && 32 * q >= BM + BN / 2)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(desc_u, dst, 16, off, kw, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(desc_w, dst, 16, off, kw, 0, 0);
    };

    // MFMA fragments: lane (l16, g4) reads 8 consecutive k of row l16: chunk 4*kc + g4 of the k-step's 8
    bf16x8 xf[2][MI], wf[2][NI];
    const int x_base = (wm * TM + l16) * ROWB + ((g4 ^ gm_swz(l16)) << 4);
    const int w_base = (BM + wn * TN + l16) * ROWB + ((g4 ^ gm_swz(l16)) << 4);
    auto read_frag = [&](auto r_c, auto kc_c, int slab_off) __attribute__((always_inline)) {
        constexpr int r = decltype(r_c)::value, kc = decltype(kc_c)::value;
        if constexpr (r < MI)
            xf[kc][r] = *reinterpret_cast<const bf16x8*>(gemm_lds + slab_off + (x_base ^ (kc * 64)) + r * 16 * ROWB);
        else
            wf[kc][r - MI] = *reinterpret_cast<const bf16x8*>(gemm_lds + slab_off + (w_base ^ (kc * 64)) + (r - MI) * 16 * ROWB);
    };

    // A k-step is 2 NM slots of one MFMA each: slice 0 (k 0..31), then slice 1.  Behind them, in slot order:
    //   slots 0 ..            the fragments of slice 1 are read (one per slot);
    //   slot BAR (in slice 1) wait for this wavefront's fragment reads and its loads of step t+1 (those of the NS-2
    //                         steps after it may still be in flight), then a barrier: slab t % NS has been read by
    //                         everyone and step t+1 has arrived for everyone;
    //   slots BAR+1 ..        the fragments of step t+1, slice 0 are read; the loads of step t+NS go out into slab
    //                         t % NS, one per LSP slots, the last of them during step t+1 (always before its BAR).
    // The loop runs the same code for every step: past the end the loads are out of range and the fragments are
    // read from slabs whose contents no MFMA uses.
    constexpr int BAR = NM + NM / 4;
    constexpr int RPS0 = (NR + NM - 1) / NM;                                    // reads per slot ahead of the barrier
    constexpr int RPS = (NR + 2 * NM - BAR - 2) / (2 * NM - BAR - 1);           // reads per slot behind the barrier
    constexpr int LSP = std::min(4, (2 * NM - 1) / NL);
    constexpr int FIRST = std::min(NL, (2 * NM - 2 - BAR) / LSP + 1);           // loads of step t+NS issued in step t
    static_assert(LSP >= 1 && LSP * (NL - 1) + 1 < 2 * NM, "reads and loads find their slots");
    static_assert(NS >= 2 && (NS - 2) * NL + FIRST <= 63, "the wait counter holds 63 loads");
    int nk = (K + 63) / 64, k_lo = 0;
    // K is a multiple of 32, so the last step may hold one slice only: then the chunks of its second half, which lie
    // past K but inside the descriptor, are pushed out of range
    int half_step = K % 64 != 0 ? nk - 1 : -1;
    if constexpr (EPI == GM_EPI_PART) {      // this split's k-steps: [k_lo, k_lo + nk), never empty
        const int all = nk;
        k_lo = (int)((int64_t)all * blockIdx.y / gridDim.y);
        nk = (int)((int64_t)all * (blockIdx.y + 1) / gridDim.y) - k_lo;
        if (half_step >= 0) half_step -= k_lo;
    }
    auto k_off = [&](int t, unsigned rec) __attribute__((always_inline)) {
        return t < nk ? (unsigned)(k_lo + t) * 128u : rec;
    };
    auto k_past = [&](int t) __attribute__((always_inline)) {
        return t == half_step && chunk >= 64 ? 0xFFFFFF00u : 0u;
    };
    auto step = [&](int t, int slab_off, int next_off, int prev_off) __attribute__((always_inline)) {
        const unsigned px = k_off(t - 1 + NS, rec_x), pw = k_off(t - 1 + NS, rec_w);
        const unsigned cx = k_off(t + NS, rec_x), cw = k_off(t + NS, rec_w);
        const unsigned p_past = k_past(t - 1 + NS), c_past = k_past(t + NS);
        static_for<2 * NM>([&](auto slot) __attribute__((always_inline)) {
            constexpr int s = decltype(slot)::value;
            constexpr int kc = s / NM, i = s % NM / MI, j = s % MI;
            asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                         : "+a"(acc[i][j]) : "v"(wf[kc][i]), "v"(xf[kc][j]));
            if constexpr (s < NM)
                static_for<RPS0>([&](auto e) __attribute__((always_inline)) {
                    constexpr int r = s * RPS0 + decltype(e)::value;
                    if constexpr (r < NR)
                        read_frag(std::integral_constant<int, r>{}, std::integral_constant<int, 1>{}, slab_off);
                });
            constexpr int late = s + 2 * NM - BAR - 1;           // slots since the barrier of the step before
            if constexpr (s < BAR && late % LSP == 0 && late / LSP >= FIRST && late / LSP < NL)
                issue_load(std::integral_constant<int, late / LSP>{}, prev_off, px, pw, p_past);
            if constexpr (s == BAR) {
                // (a plain s_barrier: __syncthreads would also drain the younger steps' loads)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * NL) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if constexpr (s > BAR) {
                static_for<RPS>([&](auto e) __attribute__((always_inline)) {
                    constexpr int r = (s - BAR - 1) * RPS + decltype(e)::value;
                    if constexpr (r < NR)
                        read_frag(std::integral_constant<int, r>{}, std::integral_constant<int, 0>{}, next_off);
                });
                if constexpr ((s - BAR - 1) % LSP == 0 && (s - BAR - 1) / LSP < FIRST)
                    issue_load(std::integral_constant<int, (s - BAR - 1) / LSP>{}, slab_off, cx, cw, c_past);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    static_for<NS>([&](auto i) __attribute__((always_inline)) {
        static_for<decltype(i)::value == NS - 1 ? FIRST : NL>([&](auto q) __attribute__((always_inline)) {
            constexpr int st = decltype(i)::value;
            issue_load(q, st * SLAB, k_off(st, rec_x), k_off(st, rec_w), k_past(st));
        });
    });
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * NL + FIRST) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<NR>([&](auto r) __attribute__((always_inline)) { read_frag(r, std::integral_constant<int, 0>{}, 0); });
    // (the asm MFMAs are opaque to the compiler's hazard rules: the accumulators were written by vector moves)
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    int slab_off = 0, prev_off = (NS - 1) * SLAB;
    int t = 0;
    do {                             // (K >= 32, and no split is empty: at least one step)
        const int next_off = slab_off + SLAB == NS * SLAB ? 0 : slab_off + SLAB;
        step(t, slab_off, next_off, prev_off);
        prev_off = slab_off;
        slab_off = next_off;
    } while (++t < nk);
    // no load may outlive the workgroup's LDS use; the last MFMAs' results may be read after their passes
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // In the accumulators a lane owns row m = .. + l16 and the 4-element column runs n = .. + 16 i + 4 g4 + r.
    if constexpr (EPI == GM_EPI_PART) {
#pragma unroll
        for (int j = 0; j < MI; ++j) {
            const int m = m0 + wm * TM + j * 16 + l16;
            if (m >= M) continue;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int n = n0 + wn * TN + i * 16 + 4 * g4;
                if (n >= N) continue;            // N % 4 == 0: the run of 4 is all in or all out
                *reinterpret_cast<f32x4*>(dist + (int64_t)m * dist_stride + n) = acc[i][j];
            }
        }
        return;
    }
    if constexpr (EPI == GM_EPI_DIST) {
#pragma unroll
        for (int j = 0; j < MI; ++j) {
            const int m = m0 + wm * TM + j * 16 + l16;
            if (m >= M) continue;
            const float sm = xsq[m];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int n = n0 + wn * TN + i * 16 + 4 * g4;
                if (n >= N) continue;
                // wsq and the rows of dist are padded to a multiple of 4 entries, so the run
                // of 4 may be read and written whole even when N cuts it
                const float4 sn = *reinterpret_cast<const float4*>(wsq + n);
                float4 o;
                o.x = __builtin_sqrtf(fmaxf(0.f, fmaf(-2.f, acc[i][j][0], sm + sn.x)));
                o.y = __builtin_sqrtf(fmaxf(0.f, fmaf(-2.f, acc[i][j][1], sm + sn.y)));
                o.z = __builtin_sqrtf(fmaxf(0.f, fmaf(-2.f, acc[i][j][2], sm + sn.z)));
                o.w = __builtin_sqrtf(fmaxf(0.f, fmaf(-2.f, acc[i][j][3], sm + sn.w)));
                *reinterpret_cast<float4*>(dist + (int64_t)m * dist_stride + n) = o;
            }
        }
        return;
    }
    // Epilogue.  Stored directly, every store instruction would touch 16 rows with 32 bytes each, and the
    // L2 request rate of all CUs finishing a round together becomes the bottleneck.  So the rounded tile
    // goes through LDS (the slab ring is free now): each wavefront stages its own TM x TN block, rows padded
    // by 16 bytes, and writes it out with 16 bytes per lane, consecutive lanes along a row.  The residual is
    // added and the norm partial is formed on the way in, in the accumulator layout.
    constexpr int STAGE_ROW = TN * 2 + 16;                // bytes; the pad spreads the rows over the banks
    __builtin_amdgcn_s_barrier();                         // every wavefront is done reading the slabs
    char* stage = gemm_lds + wv * (TM * STAGE_ROW);
#pragma unroll
    for (int j = 0; j < MI; ++j) {
        const int m = m0 + wm * TM + j * 16 + l16;
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int n = n0 + wn * TN + i * 16 + 4 * g4;
            float c[4];              // (read here and not ahead: the allocator would copy and spill the whole tile)
#pragma unroll
            for (int r = 0; r < 4; ++r) asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(c[r]) : "a"(acc[i][j][r]));
            if (EPI == GM_EPI_BF16 && res) {
                if (m < M && n < N) {            // N % 4 == 0: the run of 4 is all in or all out
                    const uint2 rr = *reinterpret_cast<const uint2*>(res + (int64_t)m * res_stride + n);
                    c[0] += bf16_lo(rr.x); c[1] += bf16_hi(rr.x);
                    c[2] += bf16_lo(rr.y); c[3] += bf16_hi(rr.y);
                }
            }
            uint2 pk;
            pk.x = pack_bf16(c[0], c[1]);
            pk.y = pack_bf16(c[2], c[3]);
            *reinterpret_cast<uint2*>(stage + (j * 16 + l16) * STAGE_ROW + (i * 16 + 4 * g4) * 2) = pk;
            if constexpr (TN == GM_PART) {
                if (sumsq_parts && n < N) {      // squares of the ROUNDED outputs, two per instruction
                    const bf16x2 lo = __builtin_bit_cast(bf16x2, pk.x), hi = __builtin_bit_cast(bf16x2, pk.y);
                    ss = __builtin_amdgcn_fdot2_f32_bf16(lo, lo, ss, false);
                    ss = __builtin_amdgcn_fdot2_f32_bf16(hi, hi, ss, false);
                }
            }
        }
        if constexpr (TN == GM_PART) {           // one partial per wavefront; other layouts never get sumsq_parts
            if (sumsq_parts) {
                ss += __shfl_xor(ss, 16, 64);
                ss += __shfl_xor(ss, 32, 64);
                const int part = (n0 + wn * TN) / GM_PART;
                if (g4 == 0 && m < M && n0 + wn * TN < N) sumsq_parts[(int64_t)part * M + m] = ss;
            }
        }
        __builtin_amdgcn_sched_barrier(0);       // one row block's residual at a time: registers
    }
    if constexpr (EPI == GM_EPI_GATED) {
        // gate block of these rows: staged by wavefront (wm, 0); up block: by (wm, 1).  Each of the two takes
        // half of the block's columns: 16-byte chunks of gate and up in, one chunk of silu(gate) * up out.
        static_assert((BN / 2) % 32 == 0, "whole loads per half");
        __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0): this wavefront's staging writes are done
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const char* gate_stage = gemm_lds + wm * (TM * STAGE_ROW);
        const char* up_stage = gemm_lds + (wm + WAVES_M) * (TM * STAGE_ROW);
        constexpr int HALF_LANES = TN / 16;               // 16-byte chunks per half row
        constexpr int ROWS_PER_PASS = 64 / HALF_LANES;    // (96-column blocks: 10 rows, the last 4 lanes idle)
        const int hrow = lane / HALF_LANES, hchunk = lane % HALF_LANES + wn * HALF_LANES;
        const int nn = n0 + hchunk * 8;
        if (nn < N && hrow < ROWS_PER_PASS) {             // N % 8 == 0: the chunk is all in or all out
#pragma unroll
            for (int r0 = 0; r0 < TM; r0 += ROWS_PER_PASS) {
                const int row = r0 + hrow;
                if (TM % ROWS_PER_PASS != 0 && row >= TM) break;
                const int m = m0 + wm * TM + row;
                const u32x4 gv = *reinterpret_cast<const u32x4*>(gate_stage + row * STAGE_ROW + hchunk * 16);
                const u32x4 uv = *reinterpret_cast<const u32x4*>(up_stage + row * STAGE_ROW + hchunk * 16);
                u32x4 ov;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g0 = bf16_lo(gv[e]), g1 = bf16_hi(gv[e]);
                    const float s0 = g0 / (1.0f + __expf(-g0)), s1 = g1 / (1.0f + __expf(-g1));
                    ov[e] = pack_bf16(s0 * bf16_lo(uv[e]), s1 * bf16_hi(uv[e]));
                }
                if (m < M) *reinterpret_cast<u32x4*>(y + (int64_t)m * y_stride + nn) = ov;
            }
        }
        return;
    }
    // (a wavefront reads back only what it wrote itself: no barrier, the LDS counter suffices)
    constexpr int LANES_PER_ROW = TN / 8;                 // 16-byte chunks per staged row
    constexpr int ROWS_PER_STORE = 64 / LANES_PER_ROW;
    const int srow = lane / LANES_PER_ROW, schunk = lane % LANES_PER_ROW;
    const int n = n0 + wn * TN + schunk * 8;
    if (n < N && srow < ROWS_PER_STORE) {                 // N % 8 == 0: the chunk is all in or all out
#pragma unroll
        for (int r0 = 0; r0 < TM; r0 += ROWS_PER_STORE) {
            const int row = r0 + srow;
            if (TM % ROWS_PER_STORE != 0 && row >= TM) break;
            const int m = m0 + wm * TM + row;
            const u32x4 val = *reinterpret_cast<const u32x4*>(stage + row * STAGE_ROW + schunk * 16);
            if (m < M) *reinterpret_cast<u32x4*>(y + (int64_t)m * y_stride + n) = val;
        }
    }
#endif
}

int gemm_sumsq_parts(int N) { return (N + GM_PART - 1) / GM_PART; }

// (as many slabs as fit in LDS, up to four)
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int NS = std::min(4, 160 * 1024 / ((BM + BN) * 128))>
static int launch_gemm_cfg(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y,
                           int64_t y_stride, const uint16_t* res, int64_t res_stride, int M, int N,
                           int K, float* sumsq_parts, const uint16_t* w2, uint16_t* y2, int n_split,
                           hipStream_t s, int64_t w_stride = 0, const float* xsq = nullptr,
                           const float* wsq = nullptr, float* dist = nullptr, int64_t dist_stride = 0,
                           int batch = 1, int64_t x_batch = 0, int64_t sq_batch = 0, int64_t dist_batch = 0) {
    if (w_stride == 0) w_stride = K;
    auto kern = gemm_kernel<BM, BN, WAVES_M, WAVES_N, EPI, NS>;
    constexpr size_t lds = gemm_lds_bytes<BM, BN, WAVES_M, WAVES_N, NS>();
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static std::atomic<bool> attr_set{false};   // per kernel instantiation; a second thread repeating the call is harmless
    if (!attr_set.load(std::memory_order_acquire)) {
        int rc = hip_status(hipFuncSetAttribute((const void*)kern,
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds),
                            "hipFuncSetAttribute(gemm)");
        if (rc) return rc;
        attr_set.store(true, std::memory_order_release);
    }
    const int tiles_m = (M + BM - 1) / BM;
    const int tiles_n = EPI == GM_EPI_GATED ? (N + BN / 2 - 1) / (BN / 2) : (N + BN - 1) / BN;
    // tile rows per group: a patch of about 32 tiles (one XCD's worth of workgroups) near square
    int group_m = 1;
    while (group_m * 2 <= tiles_m && group_m * group_m * 2 <= 32) group_m *= 2;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n, batch), dim3(GM_THREADS), lds, s, x, x_stride, w, y,
                       y_stride, res, res_stride, M, N, K, sumsq_parts, tiles_m, tiles_n, group_m, w2,
                       y2, n_split, w_stride, xsq, wsq, dist, dist_stride, x_batch, sq_batch, dist_batch);
    return launch_status("gemm");
}

// Tile shapes.  The wavefront tile sets the LDS bytes read per MFMA, so big tiles are the
// efficient ones; smaller ones exist to fill all 256 CUs when there are few rows, and the heights
// between them so that the rows of a launch end near the end of a round (2536 x 4096: 16 x 16 tiles
// of 160 x 256 are one round; 192-row tiles fill 224 of the 256 CUs).  `rate` is the measured
// throughput of a CU on that shape relative to 256x256 (K = 4096, two and three full rounds, random
// operands: 98, 85.5, 76, 65, 55, 44, 38.7, 32.6, 33.5 us a round in the order below; 160x256 and
// 224x256 against the next larger shape in use before: 2536x4096x11008 222 -> 174 us, 2536x4096x4096
// 82 -> 67 us).
struct TileShape {
    int bm, bn;
    float rate;
    bool sumsq;        // wavefront tile is 128 columns wide: can emit the norm partials
};
enum TileId { T256x256, T224x256, T192x256, T160x256, T256x128, T192x128, T160x128, T128x128, T128x128R, T128x32,
              T192x192G, T160x192G, T_COUNT };
static const TileShape kTiles[T_COUNT] = {
    {256, 256, 1.00f, true},  {224, 256, 1.00f, true},  {192, 256, 0.96f, true},  {160, 256, 0.94f, true},
    {256, 128, 0.89f, false}, {192, 128, 0.83f, false}, {160, 128, 0.79f, false}, {128, 128, 0.75f, false},
    {128, 128, 0.73f, true},  {128, 32, 0.0f, false},
    // gate/up launches only (96 gate + 96 up columns): their epilogue exists in that form alone
    {192, 192, 0.91f, false}, {160, 192, 0.88f, false},
};
constexpr float GM_TILE_US = 98.0f / 4096.0f;      // microseconds per k of a 256x256 tile

// Estimated time of the launch in units of (one 256x256 tile at full rate): rounds over the
// 256 CUs times the time of one tile.
static float tile_cost(const TileShape& t, int M, int N) {
    const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    const long rounds = (tiles + 255) / 256;
    return (float)rounds * (float)(t.bm * t.bn) / (65536.0f * t.rate);
}

// Few rows and no norm output: the weight matrix dominates the traffic and one CU cannot pull
// its share fast enough, so the columns are cut into 32-wide tiles to put every CU to work.
static bool prefer_skinny_tiles(int M, int N, int K) {
    const long mid = (long)((M + 127) / 128) * ((N + 127) / 128);
    return mid <= 64 && K % 64 == 0 && N % 32 == 0;
}

static TileId choose_tile(int M, int N, int K, bool need_sumsq, int align_n) {
    if (!need_sumsq && prefer_skinny_tiles(M, N, K)) return T128x32;
    TileId best = need_sumsq ? T128x128R : T128x128;
    float best_cost = tile_cost(kTiles[best], M, N);
    for (int i = 0; i < T128x32; ++i) {
        const TileShape& t = kTiles[i];
        if (need_sumsq && !t.sumsq) continue;
        if (align_n % t.bn != 0) continue;           // a tile must not straddle the two outputs of a pair
        const float c = tile_cost(t, M, N);
        if (c < best_cost) {
            best_cost = c;
            best = (TileId)i;
        }
    }
    return best;
}

// A launch whose tiles overflow whole rounds over the 256 CUs by a few (640 rows x 22016 columns: 3 x 86 =
// 258 tiles of 256 x 256) would spend a whole extra round on them.  Then only the leading columns, as many
// column tiles as fill the whole rounds, go out on the big tiles, and the few trailing columns follow as a
// launch of their own on the few-row / split-K path, which spreads them over the chip.  Returns the number
// of leading columns (N: no cut) and, in `id`, the tile shape for them.  A small tail (at most 64 tiles'
// worth) is priced at 0.3 of a 256 x 256 tile time (its launch and its reduction); a larger one goes out on
// whichever tile shape suits its own size and is priced as that launch plus the boundary between the two
// (5120 x 4096: 320 tiles of 256 x 256 are 1.25 rounds; 240 of them and then 160 tiles of 256 x 128 are
// one round each at their rates, 1.57 tile times instead of 2).
constexpr int GM_TAIL_MAX_TILES = 64;
constexpr float GM_TAIL_BOUNDARY = 0.08f;
static float plain_cost(int M, int N, bool need_sumsq, int align_n) {
    float best = 1e30f;
    for (int i = 0; i < T128x32; ++i) {
        const TileShape& t = kTiles[i];
        if (need_sumsq && !t.sumsq) continue;
        if (align_n % t.bn != 0) continue;
        best = std::min(best, tile_cost(t, M, N));
    }
    return best;
}
static int main_columns(TileId& id, int M, int N, int K, bool need_sumsq, int align_n, float* cost_out = nullptr) {
    if (id == T128x32) return N;
    float best = tile_cost(kTiles[id], M, N);
    int best_n = N;
    struct Report {              // the cost of the plan that is returned
        float* out;
        const float& v;
        ~Report() { if (out) *out = v; }
    } report{cost_out, best};
    for (int i = 0; i < T128x32; ++i) {
        const TileShape& t = kTiles[i];
        if (need_sumsq && !t.sumsq) continue;
        if (align_n % t.bn != 0) continue;
        const int tiles_m = (M + t.bm - 1) / t.bm, tiles_n = (N + t.bn - 1) / t.bn;
        const int rounds = (tiles_m * tiles_n + 255) / 256;
        if (rounds < 2) continue;
        const int keep_n = (rounds - 1) * 256 / tiles_m;              // column tiles that fill the whole rounds
        if (keep_n < 1 || keep_n >= tiles_n) continue;
        const bool small_tail = (tiles_n - keep_n) * tiles_m <= GM_TAIL_MAX_TILES;
        // (a large tail is priced as a plain launch: with at most 1024 rows it would be cut into k-slices instead;
        // and the tail of a pair must start where the second matrix does, or stay inside it: it is one launch)
        if (!small_tail && (M <= 1024 || (align_n != 768 && keep_n * t.bn < align_n))) continue;
        const float tail = small_tail ? 0.3f
                                      : plain_cost(M, N - keep_n * t.bn, need_sumsq, 768) + GM_TAIL_BOUNDARY;
        const float c = (float)(rounds - 1) * (float)(t.bm * t.bn) / (65536.0f * t.rate) + tail;
        if (c < best) {
            best = c;
            best_n = keep_n * t.bn;
            id = (TileId)i;
        }
    }
    return best_n;
}

static int launch_tile(TileId id, const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y,
                       int64_t y_stride, const uint16_t* res, int64_t res_stride, int M, int N, int K,
                       float* sumsq_parts, const uint16_t* w2, uint16_t* y2, int n_split, hipStream_t s) {
#define VITCOP_TILE(BM, BN, WM, WN) \
    return launch_gemm_cfg<BM, BN, WM, WN, GM_EPI_BF16>(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, \
                                                      sumsq_parts, w2, y2, n_split, s)
    switch (id) {
        case T256x256: VITCOP_TILE(256, 256, 2, 2);
        case T224x256: VITCOP_TILE(224, 256, 2, 2);
        case T192x256: VITCOP_TILE(192, 256, 2, 2);
        case T160x256: VITCOP_TILE(160, 256, 2, 2);
        case T256x128: VITCOP_TILE(256, 128, 2, 2);
        case T192x128: VITCOP_TILE(192, 128, 2, 2);
        case T160x128: VITCOP_TILE(160, 128, 2, 2);
        case T128x128: VITCOP_TILE(128, 128, 2, 2);
        case T128x128R: VITCOP_TILE(128, 128, 4, 1);
        default:
            return launch_gemm_cfg<128, 32, 4, 1, GM_EPI_BF16>(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, sumsq_parts,
                                                      w2, y2, n_split, s);
    }
#undef VITCOP_TILE
}

int launch_gemm(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y,
                int64_t y_stride, const uint16_t* res, int64_t res_stride, int M, int N,
                int K, float* sumsq_parts, hipStream_t s) {
    if (M == 0 || N == 0) return VITCOP_OK;
    const TileId id = choose_tile(M, N, K, sumsq_parts != nullptr, 768 /* any tile width divides it */);
    return launch_tile(id, x, x_stride, w, y, y_stride, res, res_stride, M, N, K, sumsq_parts, nullptr,
                       nullptr, 0, s);
}

// Two projections of the same input in one launch: y1 = x W1^T [M,N1], y2 = x W2^T [M,N2].
// Both outputs are dense and the kernel takes one output row stride, so the fused launch needs
// N1 == N2, and N1 a multiple of the tile width so that no tile straddles the two outputs;
// otherwise two launches.
int launch_gemm_pair(const uint16_t* x, int64_t x_stride, const uint16_t* w1, uint16_t* y1, int N1,
                     const uint16_t* w2, uint16_t* y2, int N2, int M, int K, hipStream_t s) {
    if (M == 0) return VITCOP_OK;
    if (N1 != N2 || N1 % 128 != 0) {
        int rc = launch_gemm(x, x_stride, w1, y1, N1, nullptr, 0, M, N1, K, nullptr, s);
        if (rc) return rc;
        return launch_gemm(x, x_stride, w2, y2, N2, nullptr, 0, M, N2, K, nullptr, s);
    }
    const TileId id = choose_tile(M, N1 + N2, K, false, N1);
    return launch_tile(id, x, x_stride, w1, y1, N1, nullptr, 0, M, N1 + N2, K, nullptr, w2, y2, N1, s);
}

// Split-K for a few hundred to a thousand rows: there are then too few large tiles to fill the chip,
// and 128 x 128 tiles, which would, load twice the bytes per FLOP through a CU's load path, which is
// what bounds them.  So the tiles stay 192 or 256 rows tall and the k-range is cut into `splits` slices
// (blockIdx.y) whose fp32 partials the few-row path's reduction kernels add up.
struct SplitKPlan {
    int bm = 0, bn = 256, splits = 0;          // splits == 0: does not apply
};
static SplitKPlan splitk_plan(int M, int N, int K) {
    SplitKPlan p;
    if (M <= 256 || M > 1024 || N % 16 != 0 || K % 32 != 0) return p;
    // 128-column tiles first: for the same number of workgroups they need half the slices of the 256-column
    // tiles, i.e. half the fp32 partials to write and to add up, and at these sizes that traffic, not the
    // matrix cores, sets the time (317 x 4096 x 4096: 28 us with 2 x 32 tiles x 4 slices against 36 us with
    // 2 x 16 tiles x 8).  Rows per tile: 160, 192 or 256, whichever leaves the shorter slice per workgroup at
    // its measured rate (640 x 4096 x 4096: 24.7 us as 4 x 32 tiles of 160 rows, 27.6 us of 192 rows).
    auto slices = [&](int tiles) { return std::min(std::min(16, 256 / std::max(tiles, 1)), K / 32 / 8); };
    auto consider = [&](const TileShape& t, int least, float& best) {
        const int s = slices((M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn));
        const float c = (float)(t.bm * t.bn) / (t.rate * (float)s);
        if (s < least || c >= best) return;
        best = c;
        p = {t.bm, t.bn, s};
    };
    float cost = 1e30f;
    for (TileId id : {T160x128, T192x128, T256x128}) consider(kTiles[id], 2, cost);
    // (not with slices longer than 4096 of k: inside a layer the 640-row down projection, K = 11008, takes
    // 110 us as 4 x 32 tiles x 2 slices against 91 us as 3 x 16 tiles x 5)
    if (p.splits < 2 || K / p.splits > 4096) {
        p = {};
        cost = 1e30f;
        for (TileId id : {T160x256, T192x256, T256x256}) consider(kTiles[id], 3, cost);
    }
    if (p.splits == 0) return p;
    // against one launch of whole tiles that needs no second pass: the partials are written and read once at
    // about 4.5 TB/s, and the reduction costs a launch (920 x 4096 x 4096: 33 us on 8 x 32 tiles of 128 x 128
    // against 33 + 13 us in two slices)
    const float split_us = cost / 65536.0f * (float)K * GM_TILE_US + 3.0f + (float)p.splits * (float)M * (float)N * 8.0f / 4.5e6f;
    float whole = 1e30f;
    for (int i = 0; i < T128x128R; ++i) whole = std::min(whole, tile_cost(kTiles[i], M, N));
    if (whole * (float)K * GM_TILE_US < split_us) p = {};
    return p;
}
static size_t splitk_workspace_bytes(int M, int N, int K) {
    const SplitKPlan p = splitk_plan(M, N, K);
    return p.splits ? up256((size_t)p.splits * M * N * 4) : 0;
}

// scratch of the trailing columns when main_columns cuts the launch (as one matrix, or as the pair N/2 + N/2)
static size_t tail_workspace_bytes(int M, int N, int K) {
    size_t need = 0;
    for (int pair = 0; pair < 2; ++pair) {
        if (pair && N % 256 != 0) break;
        for (int sumsq = 0; sumsq < (pair ? 1 : 2); ++sumsq) {
            TileId id = choose_tile(M, N, K, sumsq != 0, pair ? N / 2 : 768);
            const int n_main = main_columns(id, M, N, K, sumsq != 0, pair ? N / 2 : 768);
            if (n_main < N)
                need = std::max(need, std::max(gemm_skinny_workspace_bytes(M, N - n_main, K),
                                               splitk_workspace_bytes(M, N - n_main, K)));
        }
    }
    return need;
}

size_t gemm_workspace_bytes(int M, int N, int K) {
    const size_t whole = std::max(gemm_skinny_workspace_bytes(M, N, K), splitk_workspace_bytes(M, N, K));
    return whole ? whole : tail_workspace_bytes(M, N, K);
}

// y = x W^T (+ res) by split-K (splitk_plan applies, ws holds splitk_workspace_bytes); optionally the
// norm side output or the RMSNorm of the finished rows, as in the few-row path.
static int launch_gemm_splitk(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y, int64_t y_stride,
                              const uint16_t* res, int64_t res_stride, int M, int N, int K, float* sumsq_parts,
                              void* ws, hipStream_t s, const uint16_t* ln_w, float eps, uint16_t* norm_out,
                              int64_t norm_stride, const uint16_t* w2 = nullptr, uint16_t* y2 = nullptr,
                              int n_split = 0, SkParts* parts_out = nullptr) {
    const SplitKPlan p = splitk_plan(M, N, K);
    float* part = static_cast<float*>(ws);
    int rc;
#define VITCOP_SPLITK(BM, BN)                                                                                    \
    rc = launch_gemm_cfg<BM, BN, 2, 2, GM_EPI_PART>(x, x_stride, w, nullptr, 0, nullptr, 0, M, N, K, nullptr, w2,   \
                                                  nullptr, n_split, s, K, nullptr, nullptr, part, N, p.splits, 0, 0, \
                                                  (int64_t)M * N)
    if (p.bm == 256 && p.bn == 256) VITCOP_SPLITK(256, 256);
    else if (p.bm == 192 && p.bn == 256) VITCOP_SPLITK(192, 256);
    else if (p.bn == 256) VITCOP_SPLITK(160, 256);
    else if (p.bm == 256) VITCOP_SPLITK(256, 128);
    else if (p.bm == 192) VITCOP_SPLITK(192, 128);
    else VITCOP_SPLITK(160, 128);
#undef VITCOP_SPLITK
    if (rc) return rc;
    const SkParts parts{part, 0, p.splits, N, M};
    if (parts_out) {                             // the caller finishes the rows itself
        *parts_out = parts;
        return VITCOP_OK;
    }
    const SkMats mats{{w, w2 ? w2 : w, w}, {y, w2 ? y2 : y, y}, {y_stride, y_stride, y_stride},
                      {w2 ? n_split : N, N, N}};
    return launch_partial_reduce(parts, N, mats, res, res_stride, sumsq_parts, ln_w, eps, norm_out, norm_stride,
                                 nullptr, s);
}

int launch_gemm_ws(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y, int64_t y_stride,
                   const uint16_t* res, int64_t res_stride, int M, int N, int K, float* sumsq_parts, void* ws,
                   size_t ws_bytes, hipStream_t s) {
    if (M == 0 || N == 0) return VITCOP_OK;
    // one to four rows: a stream over W with no partial sums to reduce
    if (!sumsq_parts && gemv_applies(M, K) && N % 2 == 0 && x_stride % 8 == 0 && y_stride % 2 == 0 &&
        (!res || res_stride % 2 == 0))
        return launch_gemv(x, x_stride, nullptr, 0.f, w, y, y_stride, res, res_stride, M, N, K, s);
    const size_t need = gemm_skinny_workspace_bytes(M, N, K);
    if (ws && need && ws_bytes >= need)
        return launch_gemm_skinny(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, sumsq_parts, nullptr,
                                  nullptr, 0, ws, s);
    const size_t need_k = splitk_workspace_bytes(M, N, K);
    if (ws && need_k && ws_bytes >= need_k)
        return launch_gemm_splitk(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, sumsq_parts, ws, s, nullptr,
                                  0.f, nullptr, 0);
    if (ws) {               // a few tiles over whole rounds: leading columns on the big tiles, the rest on their own
        TileId id = choose_tile(M, N, K, sumsq_parts != nullptr, 768);
        const int n_main = main_columns(id, M, N, K, sumsq_parts != nullptr, 768);
        const size_t need_tail = n_main < N ? std::max(gemm_skinny_workspace_bytes(M, N - n_main, K),
                                                       splitk_workspace_bytes(M, N - n_main, K))
                                            : 0;
        if (n_main < N && ws_bytes >= need_tail) {
            int rc = launch_tile(id, x, x_stride, w, y, y_stride, res, res_stride, M, n_main, K, sumsq_parts, nullptr,
                                 nullptr, 0, s);
            if (rc) return rc;
            return launch_gemm_ws(x, x_stride, w + (int64_t)n_main * K, y + n_main, y_stride,
                                  res ? res + n_main : nullptr, res_stride, M, N - n_main, K,
                                  sumsq_parts ? sumsq_parts + (int64_t)(n_main / GM_PART) * M : nullptr, ws, ws_bytes, s);
        }
    }
    return launch_gemm(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, sumsq_parts, s);
}

int launch_gemm_norm_ws(const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y, int64_t y_stride,
                        const uint16_t* res, int64_t res_stride, int M, int N, int K, const uint16_t* ln_w,
                        float eps, uint16_t* norm_out, int64_t norm_stride, void* ws, size_t ws_bytes,
                        hipStream_t s) {
    if (M == 0 || N == 0) return VITCOP_OK;
    const size_t need = gemm_skinny_workspace_bytes(M, N, K);
    if (ws && need && ws_bytes >= need && gemm_skinny_fuses_norm(M, N, K))
        return launch_gemm_skinny(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, nullptr, nullptr, nullptr, 0,
                                  ws, s, ln_w, eps, norm_out, norm_stride);
    const size_t need_k = splitk_workspace_bytes(M, N, K);
    if (ws && need_k && ws_bytes >= need_k && partial_reduce_fuses_norm(N))
        return launch_gemm_splitk(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, nullptr, ws, s, ln_w, eps,
                                  norm_out, norm_stride);
    int rc = launch_gemm_ws(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, nullptr, ws, ws_bytes, s);
    if (rc) return rc;
    return launch_rmsnorm(y, y_stride, ln_w, eps, norm_out, norm_stride, M, N, s);
}

// out = silu(x Wg^T) * (x Wu^T) as ONE launch of the big tiles: a tile's columns are half gate, half up, and the
// epilogue applies the activation (GM_EPI_GATED), so gate and up never reach memory.
// (F columns of an output whose rows are out_stride apart)
static int launch_tile_gated(TileId id, const uint16_t* x, int64_t x_stride, const uint16_t* wg, const uint16_t* wu,
                             uint16_t* out, int64_t out_stride, int M, int F, int K, hipStream_t s) {
#define VITCOP_GATED(BM, BN) \
    return launch_gemm_cfg<BM, BN, 2, 2, GM_EPI_GATED>(x, x_stride, wg, out, out_stride, nullptr, 0, M, F, K, nullptr, \
                                                     wu, nullptr, 0, s)
    switch (id) {
        case T256x256: VITCOP_GATED(256, 256);
        case T224x256: VITCOP_GATED(224, 256);
        case T192x256: VITCOP_GATED(192, 256);
        case T160x256: VITCOP_GATED(160, 256);
        case T256x128: VITCOP_GATED(256, 128);
        case T192x128: VITCOP_GATED(192, 128);
        case T160x128: VITCOP_GATED(160, 128);
        case T192x192G: VITCOP_GATED(192, 192);
        case T160x192G: VITCOP_GATED(160, 192);
        default: VITCOP_GATED(128, 128);
    }
#undef VITCOP_GATED
}

int launch_gemm_gated_ws(const uint16_t* x, int64_t x_stride, const uint16_t* wg, const uint16_t* wu, int F,
                         uint16_t* gate, uint16_t* up, uint16_t* out, int M, int K, void* ws, size_t ws_bytes,
                         hipStream_t s) {
    if (M == 0 || F == 0) return VITCOP_OK;
    const size_t need = gemm_skinny_workspace_bytes(M, 2 * F, K);
    if (ws && need && ws_bytes >= need && F % 128 == 0)
        return launch_gemm_skinny_gated(x, x_stride, wg, wu, F, out, M, K, ws, s);
    // more rows than the few-row kernel takes: the big tiles with the activation in their epilogue, unless the
    // launch is one that gets cut into k-slices or sends a few trailing tiles down a path of their own (a few
    // hundred rows): those produce gate and up separately.  A large tail (many rows, whole rounds plus a part
    // of one) stays on this path: first the columns that fill the whole rounds, then the rest on the tiles
    // that suit it.
    if (F % 8 == 0 && splitk_plan(M, 2 * F, K).splits == 0) {
        const uint16_t *g_w = wg, *u_w = wu;
        uint16_t* o = out;
        int f_left = F;
        bool fused = true;
        while (f_left > 0) {
            TileId id = choose_tile(M, 2 * f_left, K, false, 768);
            if (id == T128x128R) id = T128x128;
            const bool first = f_left == F;              // only the whole launch may still go the separate way
            if (id > T128x128) {
                if (first) {
                    fused = false;
                    break;
                }
                id = T128x128;
            }
            TileId cut_id = id;
            float cut_cost = 0.f;
            int n_main = ws && f_left % 128 == 0 ? main_columns(cut_id, M, 2 * f_left, K, false, 768, &cut_cost)
                                                 : 2 * f_left;
            // (the 192-column tiles exist in this form only: a cut must beat them too)
            const TileId g192 = tile_cost(kTiles[T160x192G], M, 2 * f_left) < tile_cost(kTiles[T192x192G], M, 2 * f_left)
                                    ? T160x192G : T192x192G;
            if (cut_id == T128x128R || cut_cost >= tile_cost(kTiles[g192], M, 2 * f_left)) n_main = 2 * f_left;
            int f_now = f_left;
            if (n_main < 2 * f_left) {
                const TileShape& t = kTiles[cut_id];
                const int tail_tiles = (2 * f_left - n_main + t.bn - 1) / t.bn * ((M + t.bm - 1) / t.bm);
                if (tail_tiles <= GM_TAIL_MAX_TILES && first) {  // the small-tail cut: separate gate and up
                    fused = false;
                    break;
                }
                if (tail_tiles > GM_TAIL_MAX_TILES) {
                    id = cut_id;
                    f_now = n_main / 2;
                }
            } else if (tile_cost(kTiles[g192], M, 2 * f_left) < tile_cost(kTiles[id], M, 2 * f_left)) {
                // a few hundred rows leave the 256-column tiles a third of the CUs short (317 x 22016: 172
                // tiles); 192-column tiles (230 of 160 x 192: 65.5 us, of 192 x 192: 68 us) fill them
                id = g192;
            }
            int rc = launch_tile_gated(id, x, x_stride, g_w, u_w, o, F, M, f_now, K, s);
            if (rc) return rc;
            g_w += (int64_t)f_now * K;
            u_w += (int64_t)f_now * K;
            o += f_now;
            f_left -= f_now;
        }
        if (fused) return VITCOP_OK;
    }
    int rc = launch_gemm_pair_ws(x, x_stride, wg, gate, F, wu, up, F, M, K, ws, ws_bytes, s);
    if (rc) return rc;
    return launch_silu_mul(gate, up, out, (int64_t)M * F, s);
}

int launch_gemm_triple_ws(const uint16_t* x, int64_t x_stride, const uint16_t* const w[3], uint16_t* const y[3],
                          const int n[3], int M, int K, void* ws, size_t ws_bytes, hipStream_t s) {
    if (M == 0) return VITCOP_OK;
    const size_t need = gemm_skinny_workspace_bytes(M, n[0] + n[1] + n[2], K);
    if (ws && need && ws_bytes >= need && n[0] % 128 == 0 && n[1] % 128 == 0)
        return launch_gemm_skinny3(x, x_stride, w, y, n, M, K, ws, s);
    int rc = launch_gemm_ws(x, x_stride, w[0], y[0], n[0], nullptr, 0, M, n[0], K, nullptr, ws, ws_bytes, s);
    if (rc) return rc;
    return launch_gemm_pair_ws(x, x_stride, w[1], y[1], n[1], w[2], y[2], n[2], M, K, ws, ws_bytes, s);
}

int launch_gemm_pair_ws(const uint16_t* x, int64_t x_stride, const uint16_t* w1, uint16_t* y1, int N1,
                        const uint16_t* w2, uint16_t* y2, int N2, int M, int K, void* ws, size_t ws_bytes,
                        hipStream_t s) {
    if (M == 0) return VITCOP_OK;
    const size_t need = gemm_skinny_workspace_bytes(M, N1 + N2, K);
    if (ws && need && ws_bytes >= need && N1 == N2 && N1 % 128 == 0)
        return launch_gemm_skinny(x, x_stride, w1, y1, N1, nullptr, 0, M, N1 + N2, K, nullptr, w2, y2, N1, ws, s);
    const size_t need_k = splitk_workspace_bytes(M, N1 + N2, K);
    if (ws && need_k && ws_bytes >= need_k && N1 == N2 && N1 % 256 == 0)      // no tile straddles the two outputs
        return launch_gemm_splitk(x, x_stride, w1, y1, N1, nullptr, 0, M, N1 + N2, K, nullptr, ws, s, nullptr, 0.f,
                                  nullptr, 0, w2, y2, N1);
    if (ws && N1 == N2 && N1 % 128 == 0) {       // the same cut for the pair: the tail lies in the second matrix
        const int N = N1 + N2;
        TileId id = choose_tile(M, N, K, false, N1);
        const int n_main = main_columns(id, M, N, K, false, N1);
        const bool cut = n_main < N && n_main >= N1;
        const size_t need_tail = cut ? std::max(gemm_skinny_workspace_bytes(M, N - n_main, K),
                                                splitk_workspace_bytes(M, N - n_main, K))
                                     : 0;
        if (cut && ws_bytes >= need_tail) {
            int rc = launch_tile(id, x, x_stride, w1, y1, N1, nullptr, 0, M, n_main, K, nullptr, w2, y2, N1, s);
            if (rc) return rc;
            return launch_gemm_ws(x, x_stride, w2 + (int64_t)(n_main - N1) * K, y2 + (n_main - N1), N2, nullptr, 0, M,
                                  N - n_main, K, nullptr, ws, ws_bytes, s);
        }
    }
    return launch_gemm_pair(x, x_stride, w1, y1, N1, w2, y2, N2, M, K, s);
}

// Which way launch_gemm_qkv_rope_ws goes at M rows: 1 the three matrices in one few-row launch, 2 split-K of K
// and of the Q/V pair with their partial sums side by side in ws, 0 the plain sequence.
static int qkv_path(int M, int qd, int kd, int d, int K) {
    if (d != 64 && d != 128) return 0;
    if (gemm_skinny_workspace_bytes(M, kd + qd + kd, K) && kd % 128 == 0 && qd % 128 == 0) return 1;
    if (splitk_workspace_bytes(M, kd, K) && splitk_workspace_bytes(M, qd + kd, K) && qd == kd && kd % 256 == 0)
        return 2;
    return 0;
}

size_t gemm_qkv_workspace_bytes(int M, int Hq, int Hkv, int d, int K) {
    const int qd = Hq * d, kd = Hkv * d;
    size_t need = std::max(gemm_workspace_bytes(M, kd, K), gemm_workspace_bytes(M, qd + kd, K));
    need = std::max(need, gemm_workspace_bytes(M, kd + qd + kd, K));
    if (qkv_path(M, qd, kd, d, K) == 2)
        need = std::max(need, splitk_workspace_bytes(M, kd, K) + splitk_workspace_bytes(M, qd + kd, K));
    return need;
}

int launch_gemm_qkv_rope_ws(const uint16_t* x, int64_t x_stride, const uint16_t* wk, const uint16_t* wq,
                            const uint16_t* wv, uint16_t* k, uint16_t* q, uint16_t* v, int Hq, int Hkv, int d,
                            const int32_t* positions, float theta, int M, int K, void* ws, size_t ws_bytes,
                            hipStream_t s) {
    if (M == 0) return VITCOP_OK;
    const int qd = Hq * d, kd = Hkv * d;
    const uint16_t* const w3[3] = {wk, wq, wv};
    uint16_t* const y3[3] = {k, q, v};
    const int n3[3] = {kd, qd, kd};
    const int path = ws ? qkv_path(M, qd, kd, d, K) : 0;
    if (path == 1 && ws_bytes >= gemm_skinny_workspace_bytes(M, kd + qd + kd, K)) {
        SkParts parts{};
        int rc = launch_gemm_skinny3(x, x_stride, w3, y3, n3, M, K, ws, s, &parts);
        if (rc) return rc;
        if (parts.part == nullptr) return launch_rope(q, k, positions, M, Hq, Hkv, d, theta, s);   // written directly
        const QkvParts P{{parts, parts, parts}, {0, kd, kd + qd}};
        return launch_qkv_finish(P, k, q, v, Hq, Hkv, d, positions, theta, s);
    }
    const size_t need_k = splitk_workspace_bytes(M, kd, K), need_qv = splitk_workspace_bytes(M, qd + kd, K);
    if (path == 2 && ws_bytes >= need_k + need_qv) {
        SkParts pk{}, pqv{};
        int rc = launch_gemm_splitk(x, x_stride, wk, k, kd, nullptr, 0, M, kd, K, nullptr, ws, s, nullptr, 0.f, nullptr,
                                    0, nullptr, nullptr, 0, &pk);
        if (rc) return rc;
        rc = launch_gemm_splitk(x, x_stride, wq, q, qd, nullptr, 0, M, qd + kd, K, nullptr,
                                static_cast<char*>(ws) + need_k, s, nullptr, 0.f, nullptr, 0, wv, v, qd, &pqv);
        if (rc) return rc;
        const QkvParts P{{pk, pqv, pqv}, {0, 0, qd}};
        return launch_qkv_finish(P, k, q, v, Hq, Hkv, d, positions, theta, s);
    }
    const int rc = launch_gemm_triple_ws(x, x_stride, w3, y3, n3, M, K, ws, ws_bytes, s);
    if (rc) return rc;
    return launch_rope(q, k, positions, M, Hq, Hkv, d, theta, s);
}

// dist[b][i,j] = ||f_i - f_j||_2 in fp32 between the rows of each of `batch` bf16 matrices
// f [n,K] (row stride and batch stride in elements), with their squared row norms sq given.
// sq must be readable, and the rows of dist writable, up to the next multiple of 4 entries
// (dist_stride % 4 == 0; the pad holds garbage).
int launch_pairwise_dist(const uint16_t* f, int64_t row_stride, int64_t batch_stride, const float* sq,
                         int64_t sq_batch, float* dist, int64_t dist_stride, int64_t dist_batch, int n, int K,
                         int batch, hipStream_t s) {
    if (n == 0 || batch == 0) return VITCOP_OK;
    return launch_gemm_cfg<128, 128, 2, 2, GM_EPI_DIST>(f, row_stride, f, nullptr, 0, nullptr, 0, n, n, K, nullptr,
                                                      nullptr, nullptr, 0, s, row_stride, sq, sq, dist, dist_stride, batch,
                                                      batch_stride, sq_batch, dist_batch);
}

}  // namespace vitcop
