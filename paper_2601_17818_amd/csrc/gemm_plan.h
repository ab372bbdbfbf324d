// Which launches a projection goes out as: tile shape, k-slices, columns.  Arithmetic on sizes alone (no HIP), so
// that a test on the CPU can walk it.
#pragma once

#include <algorithm>
#include <cmath>

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
struct TileShape {
    int bm, bn;
    float rate;
    bool sumsq;        // wavefront tile is 128 columns wide: can emit the norm partials
};
enum TileId { T256x256, T224x256, T192x256, T160x256, T256x128, T192x128, T160x128, T128x128, T128x128R, T128x32,
              T192x192G, T160x192G, T_COUNT };
inline constexpr TileShape kTiles[T_COUNT] = {
    {256, 256, 1.00f, true},  {224, 256, 1.00f, true},  {192, 256, 0.96f, true},  {160, 256, 0.94f, true},
    {256, 128, 0.89f, false}, {192, 128, 0.83f, false}, {160, 128, 0.79f, false}, {128, 128, 0.75f, false},
    {128, 128, 0.73f, true},  {128, 32, 0.0f, false},
    // gate/up launches only (96 gate + 96 up columns): their epilogue exists in that form alone
    {192, 192, 0.91f, false}, {160, 192, 0.88f, false},
};
constexpr float GM_TILE_US = 98.0f / 4096.0f;      // microseconds per k of a 256x256 tile

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
inline SkinnyPlan skinny_plan(int M, int N, int K) {
    const int steps = K / SK_UNIT;
    SkinnyPlan best{0, 0, 1e30f};
    for (int cols : {64, 96, 128}) {
        const int tiles = (N + cols - 1) / cols;
        const int most = std::min(std::min(16, steps), skinny_scratch_columns(N, K) / N);
        for (int s = 1; s <= most; ++s) {
            const float us = skinny_us(skinny_rows(M), cols, tiles * s, (steps + s - 1) / s * SK_UNIT) +
                             (float)s * (float)M * (float)N * 12.0f / 4.5e6f;
            if (us < best.us) best = {cols, s, us};
        }
    }
    return best;
}

// Columns of a tile (half gate, half up) if the gate/up launch goes out as whole tiles with the activation in their
// epilogue, 0 if as the slices of `plan`.
inline int skinny_gated_columns(const SkinnyPlan& plan, int M, int F, int K) {
    const float us64 = skinny_us(skinny_rows(M), 64, F / 32, K), us128 = skinny_us(skinny_rows(M), 128, F / 64, K);
    if (std::min(us64, us128) > plan.us + 3.0f) return 0;        // (3 us: the reduction's launch)
    return us64 < us128 ? 64 : 128;
}

// ---- 257 to 1024 rows: k-slices -------------------------------------------------------------------------------

// Split-K for a few hundred to a thousand rows: there are then too few large tiles to fill the chip, and 128 x 128
// tiles, which would, load more bytes per FLOP.  So the tiles stay 160 to 256 rows tall and the k-range is cut into
// `splits` slices (workgroups of the same launch, gemm_kernel.h) whose fp32 partials the few-row path's reduction
// kernels add up.
struct SplitKPlan {
    int bm = 0, bn = 256, splits = 0;          // splits == 0: does not apply
    float us = 0.f;                            // estimate, of the launch of whole tiles if splits == 0
};
constexpr float GM_LAUNCH_US = 3.0f;
inline float splitk_us(float slice_cost, int M, int N, int K, int splits) {      // slice_cost: tile area / rate / slices
    return slice_cost / 65536.0f * (float)K * GM_TILE_US + 2.0f * GM_LAUNCH_US +
           (float)splits * (float)M * (float)N * 8.0f / 4.5e6f;
}
inline int splitk_slices(int tiles, int K) { return std::min(std::min(16, 256 / std::max(tiles, 1)), K / 32 / 8); }
// The best cut, whether or not it beats whole tiles (the scratch it would take is what callers provide).
inline SplitKPlan splitk_candidate(int M, int N, int K) {
    SplitKPlan p;
    if (M <= 256 || M > 1024 || N % 16 != 0 || K % 32 != 0) return p;
    // 128-column tiles first: for the same number of workgroups they need half the slices of the 256-column
    // tiles, i.e. half the fp32 partials to write and to add up, and at these sizes that traffic, not the
    // matrix cores, sets the time (317 x 4096 x 4096: 28 us with 2 x 32 tiles x 4 slices against 36 us with
    // 2 x 16 tiles x 8).  Rows per tile: 160, 192 or 256, whichever leaves the shorter slice per workgroup at
    // its measured rate (640 x 4096 x 4096: 24.7 us as 4 x 32 tiles of 160 rows, 27.6 us of 192 rows).
    auto consider = [&](const TileShape& t, int least, float& best) {
        const int s = splitk_slices((M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn), K);
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
    if (p.splits != 0) p.us = splitk_us(cost, M, N, K, p.splits);
    return p;
}
// The cut to take: none if one launch of whole tiles, which needs no second pass, takes no longer: the partials are
// written and read once at about 4.5 TB/s, and the reduction costs a launch (920 x 4096 x 4096: 33 us on 8 x 32
// tiles of 128 x 128 against 33 + 13 us in two slices).
inline SplitKPlan splitk_plan(int M, int N, int K) {
    SplitKPlan p = splitk_candidate(M, N, K);
    float whole = 1e30f;
    for (int i = 0; i < T128x128R; ++i) whole = std::min(whole, tile_cost(kTiles[i], M, N));
    whole = whole * (float)K * GM_TILE_US + GM_LAUNCH_US;
    if (p.splits == 0 || whole < p.us) {
        p = {};
        p.us = whole;
    }
    return p;
}
// K, Q and V of a layer as ONE launch of k-slices (tiles of 192 columns may hold the end of one matrix and the start
// of the next; 317 x 12288 x 4096: 2 x 64 tiles of 160 x 192 in two slices), where that beats a launch of K and one
// of the Q/V pair.
inline SplitKPlan qkv_plan(int M, int qd, int kd, int K) {
    SplitKPlan p;
    const int N = qd + 2 * kd;
    if (M <= 256 || M > 1024 || K % 32 != 0 || qd % 128 != 0 || kd % 128 != 0 || qd < 256 || kd < 256) return p;
    p.us = splitk_plan(M, kd, K).us + splitk_plan(M, qd + kd, K).us;
    for (TileId id : {T160x128, T192x128, T256x128, T160x192G, T192x192G}) {
        const TileShape& t = kTiles[id];
        const int s = splitk_slices((M + t.bm - 1) / t.bm * ((N + t.bn - 1) / t.bn), K);
        if (s < 2) continue;
        const float us = splitk_us((float)(t.bm * t.bn) / (t.rate * (float)s), M, N, K, s);
        if (us < p.us) p = {t.bm, t.bn, s, us};
    }
    return p;
}
// Which way launch_gemm_qkv_rope_ws goes at M rows: 1 the three matrices in one few-row launch, 3 in one launch of
// k-slices, 2 split-K of K and of the Q/V pair with their partial sums side by side in ws, 0 the plain sequence.
inline int qkv_path(int M, int qd, int kd, int d, int K) {
    if (d != 64 && d != 128) return 0;
    if (gemm_skinny_applies(M, kd + qd + kd, K) && kd % 128 == 0 && qd % 128 == 0) return 1;
    if (qkv_plan(M, qd, kd, K).splits) return 3;
    if (splitk_plan(M, kd, K).splits && splitk_plan(M, qd + kd, K).splits && qd % 256 == 0 && kd % 256 == 0)
        return 2;
    return 0;
}

}  // namespace vitcop
