// Which launches a projection goes out as: tile shape, k-slices, columns.  Arithmetic on sizes alone (no HIP), so
// that a test on the CPU can walk it.
#pragma once

#include <algorithm>
#include <cmath>
#include <initializer_list>

namespace vitcop {

// ---- whole tiles ----------------------------------------------------------------------------------------------

// Tile shapes.  The wavefront tile sets the LDS bytes read per MFMA, so big tiles are the
// efficient ones; smaller ones exist to fill all 256 CUs when there are few rows, and the heights
// between them so that the rows of a launch end near the end of a round (2536 x 4096: 16 x 16 tiles
// of 160 x 256 are one round; 192-row tiles fill 224 of the 256 CUs).  `rate` is the measured
// throughput of a CU on that shape relative to 256x256 (K = 4096, two and three full rounds, random
// operands: 98, 85.5, 76, 65, 55, 44, 38.7, 32.6, 33.5 us a round in the order below; 160x256 and
// 224x256 against the next larger shape in use before: 2536x4096x11008 222 -> 174 us, 2536x4096x4096
// 82 -> 67 us).
// `us` is the time of 4096 of k in a launch of at most a few rounds whose weights come from HBM (launch_us below).
struct TileShape {
    int bm, bn;
    float rate;
    bool sumsq;        // wavefront tile is 128 columns wide: can emit the norm partials
    float us;
};
enum TileId { T256x256, T224x256, T192x256, T160x256, T256x128, T192x128, T160x128, T128x128, T128x128R, T128x32,
              T192x192G, T160x192G, T_COUNT };
inline constexpr TileShape kTiles[T_COUNT] = {
    {256, 256, 1.00f, true, 80.0f},  {224, 256, 1.00f, true, 76.5f},  {192, 256, 0.96f, true, 65.9f},
    {160, 256, 0.94f, true, 61.2f},  {256, 128, 0.89f, false, 50.4f}, {192, 128, 0.83f, false, 43.3f},
    {160, 128, 0.79f, false, 39.7f}, {128, 128, 0.75f, false, 33.8f}, {128, 128, 0.73f, true, 34.6f},
    {128, 32, 0.0f, false, 16.1f},
    // gate/up launches and k-slices only (a gate/up tile holds 96 + 96 columns)
    {192, 192, 0.91f, false, 57.5f}, {160, 192, 0.88f, false, 50.0f},
};

// Estimated time of the launch in units of (one 256x256 tile at full rate): rounds over the
// 256 CUs times the time of one tile.
inline float tile_cost(const TileShape& t, int M, int N) {
    const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    const long rounds = (tiles + 255) / 256;
    return (float)rounds * (float)(t.bm * t.bn) / (65536.0f * t.rate);
}

// Few rows and no norm output: the weight matrix dominates the traffic and one CU cannot pull
// its share fast enough, so the columns are cut into 32-wide tiles to put every CU to work.
inline bool prefer_skinny_tiles(int M, int N, int K) {
    const long mid = (long)((M + 127) / 128) * ((N + 127) / 128);
    return mid <= 64 && K % 64 == 0 && N % 32 == 0;
}

inline TileId choose_tile(int M, int N, int K, bool need_sumsq, int align_n) {
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
inline float plain_cost(int M, int N, bool need_sumsq, int align_n) {
    float best = 1e30f;
    for (int i = 0; i < T128x32; ++i) {
        const TileShape& t = kTiles[i];
        if (need_sumsq && !t.sumsq) continue;
        if (align_n % t.bn != 0) continue;
        best = std::min(best, tile_cost(t, M, N));
    }
    return best;
}
inline int main_columns(TileId& id, int M, int N, int K, bool need_sumsq, int align_n, float* cost_out = nullptr) {
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
        // (a large tail is priced as a plain launch: with at most 1024 rows it would mostly be cut into k-slices instead;
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

// ---- at most 256 rows (gemm_skinny.hip) ----------------------------------------------------------------------

constexpr int SK_COLS = 128;          // columns per sum-of-squares partial
constexpr int SK_UNIT = 64;           // k-values per step (one 128-byte line per row)
constexpr int SK_MAX_ROWS = 256;
constexpr int SK_MAX_WGS = 256;       // one per CU

// From this many column groups on the columns alone keep most CUs streaming: whole tiles write their outputs
// themselves, and the partial sums and their reduction are saved.
constexpr int SK_DIRECT_GROUPS = 128;
inline bool skinny_direct(int N, bool want_sumsq) {
    return !want_sumsq && (N + SK_COLS - 1) / SK_COLS >= SK_DIRECT_GROUPS;
}

inline bool gemm_skinny_applies(int M, int N, int K) {
    return M >= 1 && M <= SK_MAX_ROWS && K % SK_UNIT == 0 && K >= 2 * SK_UNIT && N % 8 == 0;
}

// Scratch of a launch: twice 128 columns for each of the 256 workgroups (or column groups, if there are more);
// the plan below stays within it.
inline int skinny_scratch_columns(int N, int K) {
    const int groups = (N + SK_COLS - 1) / SK_COLS, total = groups * (K / SK_UNIT);
    return 2 * SK_COLS * std::max(groups, std::min(SK_MAX_WGS, total / 2));
}

// Time of one launch in microseconds.  A workgroup's step over 64 of k costs what its share of the HBM stream
// and its rows of x (from L2) take; the stream's rate is shared by the workgroups (with all 256 at work 0.095 ns
// per k and column, 5.4 TB/s; fewer draw less each than their number would allow, about as its square root),
// the rows cost 0.03 ns per k each.  Fitted to K = 4096 and 11008 at 32 to 224 rows; within 15 % of each.
// (Kernel alone, weights from HBM, against the unit-dealing kernel with register staging used before: 115 rows
// 12288x4096 31.4 -> 27.3 us, 4096x4096 15.2 -> 12.1, 4096x11008 31.0 -> 27.3, gate/up 22016x4096 58.7 + 7 for the
// reduction -> 48.2; 224 rows 45.7 -> 32.9, 20.3 -> 17.1, 44.1 -> 36.6, 76.1 + 8 -> 57.0; 64 rows 26.6 -> 24.8,
// 10.9 -> 9.9, 22.7 -> 22.3, 43.9 + 5 -> 42.3.)
inline float skinny_us(int rows, int cols, int wgs, int k) {
    const float share = std::sqrt(std::min(1.0f, (float)wgs / SK_MAX_WGS));
    const float rounds = (float)((wgs + SK_MAX_WGS - 1) / SK_MAX_WGS);
    return 3.0f + rounds * (float)k * (0.095e-3f * (float)cols * share + 0.03e-3f * (float)rows);
}
inline int skinny_rows(int M) { return (M + 31) / 32 * 32; }

struct SkinnyPlan {
    int cols, slices;
    float us;                            // of the launch and the traffic of its partial sums
};
// (A slice costs its traffic and a wait: the reduction reads the slices in order, and with few rows has too few
// wavefronts to hide that.  With the traffic alone the smallest outputs took 16 slices: 8 x 1024 x 1024 9.2 us, in four
// 7.6; 16 x 512 x 1024 9.2 and 7.7; 8 x 9216 x 8192 34.8 us in seven slices, 33.3 in three.)
inline SkinnyPlan skinny_plan(int M, int N, int K) {
    const int steps = K / SK_UNIT;
    const float add = 0.03f + 1.2f / (float)M;
    SkinnyPlan best{0, 0, 1e30f};
    for (int cols : {64, 96, 128}) {
        const int tiles = (N + cols - 1) / cols;
        const int most = std::min(std::min(16, steps), skinny_scratch_columns(N, K) / N);
        for (int s = 1; s <= most; ++s) {
            const float us = skinny_us(skinny_rows(M), cols, tiles * s, (steps + s - 1) / s * SK_UNIT) +
                             (float)s * ((float)M * (float)N * 12.0f / 4.5e6f + add);
            if (us < best.us) best = {cols, s, us};
        }
    }
    return best;
}

// Columns of a tile (half gate, half up) if the gate/up launch goes out as whole tiles with the activation in their
// epilogue, 0 if as the slices of `plan`.  Every form is one round of what its number of workgroups can draw, so the
// narrowest that needs no second round wins: 48 + 48 columns fill the chip where 64 + 64 leave a fifth to a quarter of
// it idle.  A whole layer of one head, us, in tiles of 32 + 32, 48 + 48 and 64 + 64 columns:
//   F x D          64 rows            115 rows           256 rows
//   8192 x 2048     80.2  83.4  85.5   96.5  99.2 101.5  119.3 121.8 122.8
//   11008 x 4096   132.2 118.4 120.6  155.5 139.0 145.7  208.2 177.7 178.6
//   18944 x 3584   157.6 153.4 162.8  189.7 181.3 190.3  256.3 227.6 237.8
//   14336 x 4096   141.0 148.3 133.1  166.7 176.5 156.1  221.6 230.4 192.9
inline int skinny_gated_columns(const SkinnyPlan& plan, int M, int F, int K) {
    int best = 0;
    float best_us = plan.us + 3.0f;                              // (3 us: the reduction's launch)
    for (int cols : {64, 96, 128}) {
        const float us = skinny_us(skinny_rows(M), cols, (2 * F + cols - 1) / cols, K);
        if (us <= best_us) {
            best_us = us;
            best = cols;
        }
    }
    return best;
}

// ---- 257 to 1536 rows: k-slices -------------------------------------------------------------------------------

constexpr int SPLITK_MAX_ROWS = 1536;

// Split-K for a few hundred to fifteen hundred rows: there are then too few large tiles to fill the chip, and 128 x 128
// tiles, which would, load more bytes per FLOP.  So the tiles stay 160 to 256 rows tall and the k-range is cut into
// `splits` slices (workgroups of the same launch, gemm_kernel.h) whose fp32 partials the few-row path's reduction
// kernels add up.
struct SplitKPlan {
    int bm = 0, bn = 256, splits = 0;          // splits == 0: whole tiles
    float us = 0.f;                            // estimate of what is taken
};
inline int tile_count(const TileShape& t, int M, int N) { return (M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn); }
// Microseconds of one launch, alone or in `slices` over k: a start and an end that grow with the tile (pipeline fill,
// epilogue), and rounds over its k, slower by a fifth with all CUs at work than with few and by a quarter with tiles
// full of rows than with rows past the end, which are not loaded (640 x 5120 x 5120: 128-row tiles 56 us, 576 rows
// 48).  This, the cost of partial sums and the table's `us` are one fit to 435 sizes of 257 to 1024 rows (256 to 12288
// columns, K 768 to 28672, weights from HBM) on each tile shape and up to 16 slices: 6 % rms; what it picks takes 1 %
// longer on average than the best measured.  The rates of full rounds alone, used before, priced a single round of
// whole tiles up to a sixth too low and slices at their traffic, and left the 128 x 32 tiles out (800 x 5120 x 13824:
// whole tiles 144 us, three slices 111; 576 x 512 x 3584: 14 slices 21.0 us, six to eight 17.7; 320 x 2048 x 2048:
// eight slices 22.1 us, 128 x 32 tiles 12.5).
inline float launch_us(const TileShape& t, int M, int N, int K, int slices = 1) {
    const int wgs = tile_count(t, M, N) * slices, rounds = (wgs + 255) / 256;
    const float fill = std::min(1.0f, (float)wgs / 256.0f);
    const float full = (float)M / (float)((M + t.bm - 1) / t.bm * t.bm);
    return 5.2f + 8.4f / 65536.0f * (float)(t.bm * t.bn) +
           (float)rounds * (float)K / (4096.0f * (float)slices) * t.us * (0.57f + 0.17f * fill + 0.26f * full);
}
// What a slice adds: its share of the reduction (partials written and read once, in slice order).
inline float slice_us(int M, int N) { return 0.27f + 1.02e-6f * (float)M * (float)N; }
constexpr float GM_REDUCTION_US = 1.4f;        // the reduction's launch
// Launches that only slices spare or only whole tiles spare: the RMSNorm after a projection and the rotary embedding
// (in the slices' reduction), the activation after gate and up (in the whole tiles' epilogue).
constexpr float GM_NORM_US = 4.0f, GM_ROPE_US = 5.0f;
inline float silu_us(int M, int F) { return 4.0f + (float)M * (float)F * 6.0f / 4.5e6f; }

inline int splitk_slices(int tiles, int K) { return std::min(std::min(16, 256 / std::max(tiles, 1)), K / 32 / 8); }
// The most slices a cut may take, which sets the scratch that callers provide (0: no cut): those that fill one round
// on the tiles that then have the shortest slices, 128 columns first, which need half the slices of 256.
inline int splitk_most(int M, int N, int K) {
    if (M <= 256 || M > SPLITK_MAX_ROWS || N % 16 != 0 || K % 32 != 0) return 0;
    auto shortest = [&](std::initializer_list<TileId> ids, int least) {
        int most = 0;
        float best = 1e30f;
        for (TileId id : ids) {
            const TileShape& t = kTiles[id];
            const int s = splitk_slices(tile_count(t, M, N), K);
            const float c = (float)(t.bm * t.bn) / (t.rate * (float)s);
            if (s < least || c >= best) continue;
            best = c;
            most = s;
        }
        return most;
    };
    const int most = shortest({T160x128, T192x128, T256x128}, 2);
    return most < 2 || K / most > 4096 ? shortest({T160x256, T192x256, T256x256}, 3) : most;
}
// The cheapest cut over the tiles `ids` of at most `most` slices, if it beats p.us.
inline void splitk_best(SplitKPlan& p, std::initializer_list<TileId> ids, int M, int N, int K, int most) {
    const float add = slice_us(M, N);
    for (TileId id : ids) {
        const TileShape& t = kTiles[id];
        const int fit = std::min(most, splitk_slices(tile_count(t, M, N), K));
        if (fit < 2) continue;
        // within one round the time is a / s + s add + a constant: least at sqrt(a / add), up to whole slices
        const int s0 = std::min((int)std::sqrt(0.8f * t.us * (float)K / (4096.0f * add)), fit - 1);
        for (int s = std::max(2, s0); s <= std::min(s0 + 1, fit); ++s) {
            const float us = launch_us(t, M, N, K, s) + GM_REDUCTION_US + (float)s * add;
            if (us < p.us) p = {t.bm, t.bn, s, us};
        }
    }
}
// The cut to take, if it beats one launch of the whole tiles that the launcher would pick, which needs no second pass.
// sumsq: with the norm side output; whole_extra_us: what the caller has to launch after whole tiles but not after
// slices (negative: the other way round).
// Between 1025 and SPLITK_MAX_ROWS rows whole tiles still leave a part of a round idle more often than not, and the price
// fitted to fewer rows picks well: layers of 3584 / 14336 (28 / 4 heads) at 1032, 1280 and 1520 rows 457 -> 425, 524 -> 494 and
// 558 -> 524 us; of 4096 / 11008 at 1080 and 1280 rows 462 -> 442 and 510 -> 494, from 1360 on the same; of 2048 / 5632 at 1120
// and 1440 193 -> 172 and 228 -> 216; of 1024 / 2816 at 1080 94 -> 88.  Above, cuts gain up to 2 % in some layers and lose up to 4
// in others (2272 rows of 1024 / 2816 112 -> 117).
inline SplitKPlan splitk_plan(int M, int N, int K, bool sumsq = false, float whole_extra_us = 0.f) {
    SplitKPlan p;
    p.us = launch_us(kTiles[choose_tile(M, N, K, sumsq, 768)], M, N, K) + whole_extra_us;
    splitk_best(p, {T160x128, T192x128, T256x128, T160x256, T192x256, T256x256}, M, N, K, splitk_most(M, N, K));
    return p;
}
// K, Q and V of a layer as ONE launch of k-slices (tiles of 192 columns may hold the end of one matrix and the start
// of the next), where that beats a launch of K and one of the Q/V pair.  `most`: slices that the scratch holds.
inline SplitKPlan qkv_plan(int M, int qd, int kd, int K, int most = 16) {
    SplitKPlan p;
    if (M <= 256 || M > SPLITK_MAX_ROWS || K % 32 != 0 || qd % 128 != 0 || kd % 128 != 0 || qd < 256 || kd < 256) return p;
    const SplitKPlan k = splitk_plan(M, kd, K), qv = splitk_plan(M, qd + kd, K);
    p.us = k.us + qv.us + (k.splits && qv.splits ? 0.f : GM_ROPE_US);
    splitk_best(p, {T160x128, T192x128, T256x128, T160x192G, T192x192G}, M, qd + 2 * kd, K, most);
    return p;
}
// Which way launch_gemm_qkv_rope_ws goes at M rows: 1 the three matrices in one few-row launch, 3 in one launch of
// k-slices, 2 split-K of K and of the Q/V pair with their partial sums side by side in ws, 0 the plain sequence.
inline int qkv_path(int M, int qd, int kd, int d, int K) {
    if (d != 64 && d != 128) return 0;
    if (gemm_skinny_applies(M, kd + qd + kd, K) && kd % 128 == 0 && qd % 128 == 0) return 1;
    if (qkv_plan(M, qd, kd, K).splits) return 3;
    const bool pairs = qd % 256 == 0 && kd % 256 == 0;
    return pairs && splitk_plan(M, kd, K).splits && splitk_plan(M, qd + kd, K).splits ? 2 : 0;
}

// ---- decoding steps -------------------------------------------------------------------------------------------

// Up to how many samples a decoding step goes out as streams over the weights (gemv.hip).  With four, every workgroup of the
// streams normalises and keeps four rows, and the matrix cores' launches, though more of them, are faster where K, Q and V are one
// of them, whose sums the attention adds up; where they are three launches, a launch for the rotary embedding follows and
// the streams win.  Four samples x 317 keys, us a layer, streams and matrix cores: 4096 / 11008 107.1, 98.0; 3584 / 14336 (28 / 4
// heads) 100.7, 95.3; 4096 / 14336 (32 / 8) 111.6, 104.0; 2048 / 5632 56.0, 52.8; 1024 / 2816 (16 / 4 of 64) 42.3, 36.3; but
// 1024 / 2816 (16 / 1 of 64) 42.5, 47.0; 2048 / 5632 (32 / 1 of 64) 55.6, 69.4, (24 / 3 of 64) 50.6, 63.9; 4096 / 11008 (64 / 1
// of 64) 109.1, 121.7.  With three samples the matrix cores are as fast (4096 / 11008 97.4, 97.9) or slower (2048 / 5632 47.7,
// 48.9; 1024 / 2816 34.9, 36.5).
inline int stream_samples(int qd, int kd, int d, int D) { return qkv_path(4, qd, kd, d, D) == 1 ? 3 : 4; }

}  // namespace vitcop
