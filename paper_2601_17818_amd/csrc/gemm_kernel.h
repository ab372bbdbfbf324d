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
#pragma once

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

// y = x W^T (+ residual).  Up to three weight matrices sit side by side in one launch (projections of the
// same input): SkMats says which columns belong to which and where each one's output goes.  A tile belongs to
// one matrix (their boundaries are multiples of the tile width), except for the k-sliced tiles of at most 192
// columns, which may hold the end of one and the start of the next (boundaries multiples of 32).
// EPI selects the epilogue: GM_EPI_BF16 the projection described above; GM_EPI_GRAM the inner products between the
// rows of one matrix per image (x and w are the same), in two k-slices: the products are symmetric, so the first half
// of k is summed in the tiles above the diagonal and the second half in those below it, and dist[i][j] + dist[j][i]
// is <x_i, x_j>; the two halves of the rows' sums of squares go to sumsq_parts[i] and sumsq_parts[sq_half + i].
// GM_EPI_PART is split-K: a workgroup multiplies its slice's share of the k-steps and writes the
// raw fp32 accumulators to dist[split][m][n] (row stride dist_stride, slices dist_batch apart) for a
// reduction kernel to add up.
// GM_EPI_GATED is the MLP's first half in one launch: a tile's first BN/2 columns are rows of the first matrix
// (gate), its last BN/2 the same rows of the second (up); N counts the columns of each; the epilogue rounds both to bf16 as the
// two separate projections would, and stores y[m,n] = silu(gate[m,n]) * up[m,n] (WAVES_N == 2: the gate
// columns of a tile belong to the wavefronts with wn = 0, the up columns to wn = 1).
constexpr int GM_EPI_BF16 = 0, GM_EPI_GRAM = 1, GM_EPI_PART = 2, GM_EPI_GATED = 3;

// What bounds the big tiles is the issue of MFMAs and, behind it, power: 11776x4096x4096 takes 234 us on all-zero and
// 278 us on random operands, and over both the matrix cores are busy 69 % of the launch's cycles (62 % before the
// layout below).  16x16x32 instructions (half the accumulator
// traffic per FLOP of 32x32x16) in an order fixed by sched_barrier, each pinned to accumulation registers by an
// asm constraint (left to itself the allocator moves 60 % as many registers as there are MFMAs); k-steps of 64
// (every direct load moves 8 whole lines), loads one per four or five MFMAs so that a CU's load path
// (64 bytes per clock) is never asked for more than it moves and no wavefront is stuck on issuing one.
// Against 32x32x16 with four slabs of 32 and compiler scheduling hints (GPU time, random operands, same box):
// 11776x4096x4096 354 -> 278 us (1116 -> 1424 TFLOP/s), 1536x8192x4096 107 -> 77 us.
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int NS, bool SPREAD>
__global__ __launch_bounds__(GM_THREADS) void gemm_kernel(
    const uint16_t* __restrict__ x, int64_t x_stride, SkMats mats, const uint16_t* __restrict__ res,
    int64_t res_stride, int M, int N, int K, float* __restrict__ sumsq_parts, int tiles_m,
    int tiles_n, int group_m, int64_t w_stride, float* __restrict__ dist, int64_t dist_stride, int64_t x_batch,
    int64_t sq_batch, int64_t sq_half, int64_t dist_batch) {
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
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);      // wavefront index, kept scalar
    const int l16 = lane & 15, g4 = lane >> 4;
    const int wm = wv % WAVES_M, wn = wv / WAVES_M;

    // Workgroup -> (z, tile); z is the k-slice (PART) or the image (GRAM).  Consecutive workgroup ids go to
    // different XCDs, so id % 8 picks the XCD and id / 8 the slot inside it; each XCD walks a contiguous range
    // of a grouped ordering (group_m tile rows by all tile columns, column-major inside the group), z outermost:
    // the tiles that share rows of W, and the slices that share a k-range of x, meet in one L2.
    int tile_m, tile_n, z;
    [[maybe_unused]] bool below = false;         // GRAM: a tile of the second half of k
    {
        const int nt = EPI == GM_EPI_GRAM ? tiles_m * (tiles_m + 1) : tiles_m * tiles_n;
        const int xcd = blockIdx.x % GM_XCDS;
        int lin = xcd * (gridDim.x / GM_XCDS) + min(xcd, (int)(gridDim.x % GM_XCDS)) + blockIdx.x / GM_XCDS;
        z = lin / nt;
        lin -= z * nt;
        if constexpr (EPI == GM_EPI_GRAM) {      // a list of the tiles on and above the diagonal, then of those mirrored
            below = lin >= nt / 2;
            int a = below ? lin - nt / 2 : lin, b = 0;
            while (a > b) a -= ++b;
            tile_m = below ? b : a;
            tile_n = below ? a : b;
        } else {
            const int width = group_m * tiles_n;
            const int grp = lin / width;
            const int first = grp * group_m;
            const int gsz = min(tiles_m - first, group_m);
            const int in = lin - grp * width;
            tile_m = first + in % gsz;
            tile_n = in / gsz;
        }
    }
    if constexpr (EPI == GM_EPI_PART) dist += z * dist_batch;
    if constexpr (EPI == GM_EPI_GRAM) {      // x and w are the same feature matrix
        x += z * x_batch;
        dist += z * dist_batch;
    }
    const int m0 = tile_m * BM;
    // n0, N: first column and number of columns, inside this tile's matrix (of a straddling tile: of the launch)
    int n0 = tile_n * (EPI == GM_EPI_GATED ? BN / 2 : BN);
    constexpr bool STRADDLE = EPI == GM_EPI_PART && BN < 256;
    static_assert(EPI != GM_EPI_GATED || WAVES_N == 2, "gate and up halves go to the two wavefront columns");
    const uint16_t *w = mats.w[0], *w_next = EPI == GM_EPI_GATED ? mats.w[1] : mats.w[0];
    uint16_t* y = mats.y[0];
    int64_t y_stride = mats.y_stride[0];
    int next_row = BN;               // the first tile row of W that belongs to the next matrix
    if constexpr (EPI == GM_EPI_GRAM) {
        w = w_next = mats.w[0] + z * x_batch;
    } else if constexpr (EPI == GM_EPI_GATED) {
        next_row = BN / 2;
    } else {
        const SkPick pick = sk_pick(mats, n0);
        w = mats.w[pick.mi];
        y = mats.y[pick.mi];
        y_stride = mats.y_stride[pick.mi];
        const int end = pick.mi == 2 ? N : min(mats.n_end[pick.mi], N);
        if constexpr (STRADDLE) {
            if (end < N) next_row = min(end - n0, BN);
            // (tile row r of the next matrix is its row r - next_row)
            w_next = mats.w[pick.mi == 2 ? 2 : pick.mi + 1] - (int64_t)next_row * w_stride;
            w += (int64_t)(n0 - pick.start) * w_stride;
        } else {
            n0 -= pick.start;
            N = end - pick.start;
            if constexpr (EPI == GM_EPI_PART) dist += pick.start;        // partials keep the launch's columns
        }
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
    const int rows_x = min(M - m0, BM), rows_all = min(N - n0, EPI == GM_EPI_GATED ? BN / 2 : BN);
    const int rows_w = STRADDLE ? min(rows_all, next_row) : rows_all;
    const unsigned rec_x = 2u * ((unsigned)(rows_x - 1) * (unsigned)x_stride + (unsigned)K);
    const unsigned rec_w = 2u * ((unsigned)(rows_w - 1) * (unsigned)w_stride + (unsigned)K);
    const unsigned rec_u = STRADDLE ? 2u * ((unsigned)(rows_all - 1) * (unsigned)w_stride + (unsigned)K) : rec_w;
    auto descriptor = [](const uint16_t* base, unsigned bytes) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);     // raw buffer, 32-bit data format
    };
    const auto desc_x = descriptor(x + (int64_t)m0 * x_stride, rec_x);
    const auto desc_w = descriptor(STRADDLE ? w : w + (int64_t)n0 * w_stride, rec_w);
    const auto desc_u = descriptor(STRADDLE ? w_next : w_next + (int64_t)n0 * w_stride, rec_u);
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
        if constexpr (32 * q < BM) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(desc_x, dst, 16, off, kx, 0, 0);
        } else if constexpr (STRADDLE) {
            const bool next = 32 * q - BM >= next_row;               // uniform: boundaries are multiples of 32
            __builtin_amdgcn_raw_ptr_buffer_load_lds(next ? desc_u : desc_w, dst, 16, off,
                                                     kw == rec_w && next ? rec_u : kw, 0, 0);
        } else if constexpr (EPI == GM_EPI_GATED && 32 * q < BM + BN / 2 && 32 * q + 32 > BM + BN / 2) {
            // (halves of 48 columns: two of the wavefronts hold the last gate rows, two the first up rows; rec_u == rec_w)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(32 * q + 8 * wv >= BM + BN / 2 ? desc_u : desc_w, dst, 16, off, kw, 0, 0);
        } else if constexpr (EPI == GM_EPI_GATED && 32 * q >= BM + BN / 2) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(desc_u, dst, 16, off, kw, 0, 0);
        } else {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(desc_w, dst, 16, off, kw, 0, 0);
        }
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
    // With two slabs that leaves the last loads half a step to arrive.  EARLY: a second barrier at slot REL, as soon as
    // the fragments of slice 1 have been read, releases the slab, the loads of step t+2 follow it at once, and BAR
    // moves to the end of the step, so that every load has a whole step and more (two full rounds of 256x256 201 ->
    // 195 us, of 224x256 180 -> 170, of 192x256 169 -> 150; 1536x8192x4096 86 -> 77 us; with three slabs no gain).
    // The loop runs the same code for every step: past the end the loads are out of range and the fragments are
    // read from slabs whose contents no MFMA uses.
    constexpr bool EARLY = NS == 2;
    constexpr int RPS0 = (NR + NM - 1) / NM;                                    // reads per slot ahead of the barrier
    constexpr int REL = NR / RPS0 + NM / 8;
    constexpr int BAR = EARLY ? 2 * NM - NR - NM / 8 - 1 : NM + NM / 4;
    constexpr int RPS = (NR + 2 * NM - BAR - 2) / (2 * NM - BAR - 1);           // reads per slot behind the barrier
    constexpr int LSP = EARLY ? std::min(5, (2 * NM - 2 - REL) / NL) : std::min(4, (2 * NM - 1) / NL);
    constexpr int FIRST = EARLY ? NL : std::min(NL, (2 * NM - 2 - BAR) / LSP + 1);          // loads of step t+NS issued in step t
    constexpr int YOUNGER = (NS - 2) * NL + (EARLY ? std::min(NL, (BAR - REL - 1) / LSP + 1) : 0);      // loads behind those of step t+1 at BAR
    static_assert(LSP >= 1 && LSP * (NL - 1) + 1 < 2 * NM && (!EARLY || REL + 1 + LSP * (NL - 1) < 2 * NM), "reads and loads find their slots");
    static_assert(NS >= 2 && (NS - 2) * NL + FIRST <= 63, "the wait counter holds 63 loads");
    int nk = (K + 63) / 64, k_lo = 0;
    // K is a multiple of 32, so the last step may hold one slice only: then the chunks of its second half, which lie
    // past K but inside the descriptor, are pushed out of range
    int half_step = K % 64 != 0 ? nk - 1 : -1;
    if constexpr (EPI == GM_EPI_PART) {      // this split's k-steps: [k_lo, k_lo + nk), never empty
        const int all = nk;
        const int slices = gridDim.x / (tiles_m * tiles_n);
        k_lo = (int)((int64_t)all * z / slices);
        nk = (int)((int64_t)all * (z + 1) / slices) - k_lo;
        if (half_step >= 0) half_step -= k_lo;
    }
    if constexpr (EPI == GM_EPI_GRAM) {      // the first half (K <= 64: all) or the second (K <= 64: nothing, which reads as zeros)
        const int first_half = (nk + 1) / 2;
        if (below) {
            k_lo = first_half;
            if (half_step >= 0) half_step -= k_lo;
            nk -= first_half;
        } else {
            nk = first_half;
        }
    }
    // Up to a few hundred rows a launch is a stream over W from HBM, and its workgroups, which read rows a power of two apart
    // as often as not, would in step all ask for the same few columns, i.e. for a part of the memory channels (loads alone,
    // 230 tiles of 96 columns of 4096 and 64 rows of x: 39.8 us in step, 31.2 apart).  So long slices start at different k
    // and wrap around: where one tile holds all rows, the tiles spread evenly over k; where the rows take two, the
    // eight XCDs do, and the tiles of one, which share the rows of x and of W in its L2, stay in step.  The start is a matter
    // of the columns alone, so that equal rows get equal sums wherever they stand in a launch: the two tiles of a column
    // follow each other in the XCDs' ranges, and where the second is the first of its XCD's it starts as the one before
    // does.  Layers of 4096 /
    // 11008, us each, in step / one k-step further from tile to tile (used before, up to 64 rows) / this: 64 decoding rows
    // 126.5 / 116.0 / 114.6; 32 rows 116.6 / 108.1 / 104.4; prefill of 115 rows 144.1 / 138.8 / 137.4; 317 rows
    // 204.6 / 200.0 / 199.5.  640 rows, three and four tiles, are the same either way and stay in step, and whole tiles of
    // thousands of rows, whose W comes from L2, lose 0.7 %.  Short slices stay in step (4096x4096 in four slices of 16
    // steps: 7.4 to 7.9 us for 7.5).
    // Launches of more rows are built without the wrap-around, whose addresses cost a step up to 2.5 % (2536 rows, the last
    // 1280 columns of gate and of up on tiles of 160 x 192: 57.3 -> 55.9 us).
    int rot = 0;
    if (SPREAD && nk >= 32)
        rot = tiles_m == 1 ? tile_n * nk / tiles_n
                           : ((int)(blockIdx.x % GM_XCDS) - (tile_m == 1 && blockIdx.x < GM_XCDS)) * nk / GM_XCDS;
    auto k_at = [&](int t) __attribute__((always_inline)) {
        if constexpr (!SPREAD) return t;
        return t + rot >= nk ? t + rot - nk : t + rot;
    };
    auto k_off = [&](int t, unsigned rec) __attribute__((always_inline)) {
        return t < nk ? (unsigned)(k_lo + k_at(t)) * 128u : rec;
    };
    auto k_past = [&](int t) __attribute__((always_inline)) {
        return k_at(t) == half_step && chunk >= 64 ? 0xFFFFFF00u : 0u;
    };
    // GRAM, tiles on the diagonal: the sums of squares of the tile's rows, from the slab while it is there (16 or 32
    // elements per thread and step, a sum for each pair: as many terms per sum as the half has steps, then pairwise).  The
    // diagonal of the product itself, one chain of K / 64 MFMAs per element, made the densities a sixth less accurate.
    constexpr int SQ_TPR = GM_THREADS / BM > 0 ? GM_THREADS / BM : 1, SQ_CHUNKS = EPI == GM_EPI_GRAM ? 8 / SQ_TPR : 1;
    [[maybe_unused]] float row_sq[SQ_CHUNKS][4];
    if constexpr (EPI == GM_EPI_GRAM)
#pragma unroll
        for (int c = 0; c < SQ_CHUNKS; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) row_sq[c][e] = 0.f;
    auto step = [&](int t, int slab_off, int next_off, int prev_off) __attribute__((always_inline)) {
        [[maybe_unused]] bf16x8 own_row[SQ_CHUNKS];          // (read ahead of the barrier that releases the slab)
        if constexpr (EPI == GM_EPI_GRAM)
#pragma unroll
            for (int c = 0; c < SQ_CHUNKS; ++c)
                own_row[c] = *reinterpret_cast<const bf16x8*>(gemm_lds + slab_off + tid / SQ_TPR * ROWB +
                                                              (((tid % SQ_TPR * SQ_CHUNKS + c) ^ gm_swz(tid / SQ_TPR)) << 4));
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
            if constexpr (EARLY && s == REL) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if constexpr (EARLY && s > REL && (s - REL - 1) % LSP == 0 && (s - REL - 1) / LSP < NL)
                issue_load(std::integral_constant<int, (s - REL - 1) / LSP>{}, slab_off, cx, cw, c_past);
            constexpr int late = s + 2 * NM - BAR - 1;           // slots since the barrier of the step before
            if constexpr (!EARLY && s < BAR && late % LSP == 0 && late / LSP >= FIRST && late / LSP < NL)
                issue_load(std::integral_constant<int, late / LSP>{}, prev_off, px, pw, p_past);
            if constexpr (s == BAR) {
                // (a plain s_barrier: __syncthreads would also drain the younger steps' loads)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(YOUNGER) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            if constexpr (s > BAR) {
                static_for<RPS>([&](auto e) __attribute__((always_inline)) {
                    constexpr int r = (s - BAR - 1) * RPS + decltype(e)::value;
                    if constexpr (r < NR)
                        read_frag(std::integral_constant<int, r>{}, std::integral_constant<int, 0>{}, next_off);
                });
                if constexpr (!EARLY && (s - BAR - 1) % LSP == 0 && (s - BAR - 1) / LSP < FIRST)
                    issue_load(std::integral_constant<int, (s - BAR - 1) / LSP>{}, slab_off, cx, cw, c_past);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (EPI == GM_EPI_GRAM)
            if (tile_m == tile_n)
#pragma unroll
                for (int c = 0; c < SQ_CHUNKS; ++c) {
                    const u32x4 word = __builtin_bit_cast(u32x4, own_row[c]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {        // two squares per instruction
                        const uint32_t w32 = word[e];    // (a copy: a bit cast of the vector's element takes the first one)
                        const bf16x2 two = __builtin_bit_cast(bf16x2, w32);
                        row_sq[c][e] = __builtin_amdgcn_fdot2_f32_bf16(two, two, row_sq[c][e], false);
                    }
                }
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
    if constexpr (EPI == GM_EPI_GRAM) {
#pragma unroll
        for (int j = 0; j < MI; ++j) {
            const int m = m0 + wm * TM + j * 16 + l16;
            if (m >= M) continue;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int n = n0 + wn * TN + i * 16 + 4 * g4;
                float* out = dist + (int64_t)m * dist_stride + n;
                // a run of 4 may end in the row's pad (rows are padded to a multiple of 4)
                if (tile_m != tile_n) {
                    if (n < N) *reinterpret_cast<f32x4*>(out) = acc[i][j];
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (n + r < N && (below ? n + r < m : n + r > m)) out[r] = acc[i][j][r];
                }
            }
        }
        if (tile_m == tile_n) {
            float ss = 0.f;
#pragma unroll
            for (int e = 4; e > 1; e >>= 1)              // pairwise
#pragma unroll
                for (int c = 0; c < SQ_CHUNKS; ++c)
#pragma unroll
                    for (int u = 0; u < e / 2; ++u) row_sq[c][u] += row_sq[c][u + e / 2];
#pragma unroll
            for (int c = 0; c < SQ_CHUNKS; ++c) ss += row_sq[c][0];
#pragma unroll
            for (int o = 1; o < SQ_TPR; o <<= 1) ss += __shfl_xor(ss, o, 64);
            const int m = m0 + tid / SQ_TPR;
            if (tid % SQ_TPR == 0 && m < M) sumsq_parts[(below ? sq_half : 0) + z * sq_batch + m] = ss;
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
        static_assert((BN / 2) % 16 == 0 && BN % 32 == 0, "whole rows of a load per half");
        __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0): this wavefront's staging writes are done
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const char* gate_stage = gemm_lds + wm * (TM * STAGE_ROW);
        const char* up_stage = gemm_lds + (wm + WAVES_M) * (TM * STAGE_ROW);
        constexpr int HALF_LANES = TN / 16;               // 16-byte chunks per half row
        constexpr int ROWS_PER_PASS = 64 / HALF_LANES;    // (96- and 48-column blocks: 10 and 21 rows, the last 4 and 1 lanes idle)
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

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int NS, bool SPREAD>
static int launch_gemm_as(const uint16_t* x, int64_t x_stride, const SkMats& mats, const uint16_t* res,
                          int64_t res_stride, int M, int N, int K, float* sumsq_parts,
                          hipStream_t s, int64_t w_stride, float* dist, int64_t dist_stride,
                          int batch, int64_t x_batch, int64_t sq_batch, int64_t dist_batch, int64_t sq_half) {
    auto kern = gemm_kernel<BM, BN, WAVES_M, WAVES_N, EPI, NS, SPREAD>;
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
    const int tiles = EPI == GM_EPI_GRAM ? tiles_m * (tiles_m + 1) : tiles_m * tiles_n;
    hipLaunchKernelGGL(kern, dim3(tiles * batch), dim3(GM_THREADS), lds, s, x, x_stride, mats, res,
                       res_stride, M, N, K, sumsq_parts, tiles_m, tiles_n, group_m, w_stride, dist, dist_stride, x_batch, sq_batch, sq_half, dist_batch);
    return launch_status("gemm");
}

// (as many slabs as fit in LDS, up to four; FEW: the tile always holds all rows)
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, bool FEW = false,
          int NS = std::min(4, 160 * 1024 / ((BM + BN) * 128))>
static int launch_gemm_cfg(const uint16_t* x, int64_t x_stride, const SkMats& mats, const uint16_t* res,
                           int64_t res_stride, int M, int N, int K, float* sumsq_parts,
                           hipStream_t s, int64_t w_stride = 0, float* dist = nullptr, int64_t dist_stride = 0,
                           int batch = 1, int64_t x_batch = 0, int64_t sq_batch = 0, int64_t dist_batch = 0, int64_t sq_half = 0) {
    if (w_stride == 0) w_stride = K;
    auto launch = launch_gemm_as<BM, BN, WAVES_M, WAVES_N, EPI, NS, FEW>;
    if constexpr (!FEW && (EPI == GM_EPI_PART || EPI == GM_EPI_GATED))
        if (M <= 2 * BM) launch = launch_gemm_as<BM, BN, WAVES_M, WAVES_N, EPI, NS, true>;
    return launch(x, x_stride, mats, res, res_stride, M, N, K, sumsq_parts, s, w_stride, dist, dist_stride, batch, x_batch,
                  sq_batch, dist_batch, sq_half);
}

}  // namespace vitcop
