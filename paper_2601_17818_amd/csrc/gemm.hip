// Launches of the projection kernel (gemm_kernel.h), as gemm_plan.h picks them.
#include <numeric>

#include "gemm_kernel.h"
#include "gemm_plan.h"

namespace vitcop {

int gemm_sumsq_parts(int N) { return (N + GM_PART - 1) / GM_PART; }

static int launch_tile_mats(TileId id, const uint16_t* x, int64_t x_stride, const SkMats& mats, const uint16_t* res,
                            int64_t res_stride, int M, int N, int K, float* sumsq_parts, hipStream_t s) {
#define VITCOP_TILE(BM, BN, WM, WN) \
    return launch_gemm_cfg<BM, BN, WM, WN, GM_EPI_BF16>(x, x_stride, mats, res, res_stride, M, N, K, sumsq_parts, s)
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
            return launch_gemm_cfg<128, 32, 4, 1, GM_EPI_BF16>(x, x_stride, mats, res, res_stride, M, N, K, sumsq_parts, s);
    }
#undef VITCOP_TILE
}
static int launch_tile(TileId id, const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y,
                       int64_t y_stride, const uint16_t* res, int64_t res_stride, int M, int N, int K,
                       float* sumsq_parts, const uint16_t* w2, uint16_t* y2, int n_split, hipStream_t s,
                       int64_t y2_stride = 0) {
    return launch_tile_mats(id, x, x_stride, sk_mats(w, y, y_stride, N, w2, y2, n_split, y2_stride), res, res_stride, M, N,
                            K, sumsq_parts, s);
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
// N1 must be a multiple of the tile width so that no tile straddles the two outputs; otherwise two launches.
// (755 rows, 3584 + 512 columns, K = 3584: one launch of 192 tiles instead of one of 168 and one of 24,
// 28 us instead of 35 + 15.)
int launch_gemm_pair(const uint16_t* x, int64_t x_stride, const uint16_t* w1, uint16_t* y1, int N1,
                     const uint16_t* w2, uint16_t* y2, int N2, int M, int K, hipStream_t s) {
    if (M == 0) return VITCOP_OK;
    if (N1 % 128 != 0) {
        int rc = launch_gemm(x, x_stride, w1, y1, N1, nullptr, 0, M, N1, K, nullptr, s);
        if (rc) return rc;
        return launch_gemm(x, x_stride, w2, y2, N2, nullptr, 0, M, N2, K, nullptr, s);
    }
    const TileId id = choose_tile(M, N1 + N2, K, false, N1);
    return launch_tile(id, x, x_stride, w1, y1, N1, nullptr, 0, M, N1 + N2, K, nullptr, w2, y2, N1, s, N2);
}

static size_t splitk_workspace_bytes(int M, int N, int K) { return up256((size_t)splitk_most(M, N, K) * M * N * 4); }

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

// the k-slices of p over the matrices of `mats`, into part
static int launch_slices(const SplitKPlan& p, const uint16_t* x, int64_t x_stride, const SkMats& mats, int M, int N, int K,
                         float* part, hipStream_t s) {
#define VITCOP_SPLITK(BM, BN)                                                                                          \
    return launch_gemm_cfg<BM, BN, 2, 2, GM_EPI_PART>(x, x_stride, mats, nullptr, 0, M, N, K, nullptr, s, K, part, N, \
                                                      p.splits, 0, 0, (int64_t)M * N)
    switch (p.bm * 1024 + p.bn) {
        case 256 * 1024 + 256: VITCOP_SPLITK(256, 256);
        case 192 * 1024 + 256: VITCOP_SPLITK(192, 256);
        case 160 * 1024 + 256: VITCOP_SPLITK(160, 256);
        case 192 * 1024 + 192: VITCOP_SPLITK(192, 192);
        case 160 * 1024 + 192: VITCOP_SPLITK(160, 192);
        case 256 * 1024 + 128: VITCOP_SPLITK(256, 128);
        case 192 * 1024 + 128: VITCOP_SPLITK(192, 128);
        default: VITCOP_SPLITK(160, 128);
    }
#undef VITCOP_SPLITK
}

// y = x W^T (+ res) in the k-slices of p (ws holds splitk_workspace_bytes); optionally the
// norm side output or the RMSNorm of the finished rows, as in the few-row path.
static int launch_gemm_splitk(const SplitKPlan& p, const uint16_t* x, int64_t x_stride, const uint16_t* w, uint16_t* y,
                              int64_t y_stride, const uint16_t* res, int64_t res_stride, int M, int N, int K,
                              float* sumsq_parts, void* ws, hipStream_t s, const uint16_t* ln_w, float eps,
                              uint16_t* norm_out, int64_t norm_stride, const uint16_t* w2 = nullptr,
                              uint16_t* y2 = nullptr, int n_split = 0, SkParts* parts_out = nullptr) {
    float* part = static_cast<float*>(ws);
    const SkMats mats = sk_mats(w, y, y_stride, N, w2, y2, n_split, w2 ? N - n_split : 0);
    const int rc = launch_slices(p, x, x_stride, mats, M, N, K, part, s);
    if (rc) return rc;
    const SkParts parts{part, p.splits, N, M};
    if (parts_out) {                             // the caller finishes the rows itself
        *parts_out = parts;
        return VITCOP_OK;
    }
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
    if (ws && ws_bytes >= splitk_workspace_bytes(M, N, K)) {
        const SplitKPlan p = splitk_plan(M, N, K, sumsq_parts != nullptr);
        if (p.splits)
            return launch_gemm_splitk(p, x, x_stride, w, y, y_stride, res, res_stride, M, N, K, sumsq_parts, ws, s,
                                      nullptr, 0.f, nullptr, 0);
    }
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
    if (ws && ws_bytes >= splitk_workspace_bytes(M, N, K) && partial_reduce_fuses_norm(N)) {
        const SplitKPlan p = splitk_plan(M, N, K, false, GM_NORM_US);
        if (p.splits)
            return launch_gemm_splitk(p, x, x_stride, w, y, y_stride, res, res_stride, M, N, K, nullptr, ws, s, ln_w, eps,
                                      norm_out, norm_stride);
    }
    int rc = launch_gemm_ws(x, x_stride, w, y, y_stride, res, res_stride, M, N, K, nullptr, ws, ws_bytes, s);
    if (rc) return rc;
    return launch_rmsnorm(y, y_stride, ln_w, eps, norm_out, norm_stride, M, N, s);
}

// out = silu(x Wg^T) * (x Wu^T) as ONE launch of the big tiles: a tile's columns are half gate, half up, and the
// epilogue applies the activation (GM_EPI_GATED), so gate and up never reach memory.
// (F columns of an output whose rows are out_stride apart)
static int launch_tile_gated(TileId id, const uint16_t* x, int64_t x_stride, const uint16_t* wg, const uint16_t* wu,
                             uint16_t* out, int64_t out_stride, int M, int F, int K, hipStream_t s) {
    const SkMats mats{{wg, wu, wu}, {out, out, out}, {out_stride, out_stride, out_stride}, {F, F, F}};
#define VITCOP_GATED(BM, BN) \
    return launch_gemm_cfg<BM, BN, 2, 2, GM_EPI_GATED>(x, x_stride, mats, nullptr, 0, M, F, K, nullptr, s)
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
    if (F % 8 == 0 && splitk_plan(M, 2 * F, K, false, -silu_us(M, F)).splits == 0) {
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
    // many rows: whole tiles of all three in one launch, where that takes no more rounds than the first matrix and the
    // other two apart: the end of one launch and the start of the next overlap
    // (layers of 2048 / 5632 at 1200 rows, six of them: 1190 -> 1133 us; of 4096 / 11008 at 2536 rows 5437 -> 5427)
    const int N = n[0] + n[1] + n[2];
    if (M > 1024 && n[0] % 128 == 0 && n[1] % 128 == 0 && n[0] > 0 && n[1] > 0) {
        const int align = std::gcd(n[0], n[1]);
        TileId id0 = choose_tile(M, n[0], K, false, 768), id12 = choose_tile(M, n[1] + n[2], K, false, n[1]);
        float c0 = tile_cost(kTiles[id0], M, n[0]), c12 = tile_cost(kTiles[id12], M, n[1] + n[2]);
        main_columns(id0, M, n[0], K, false, 768, &c0);
        main_columns(id12, M, n[1] + n[2], K, false, n[1], &c12);
        const TileId id = choose_tile(M, N, K, false, align);
        if (id0 != T128x32 && id12 != T128x32 && id != T128x32 && tile_cost(kTiles[id], M, N) <= c0 + c12) {
            const SkMats mats{{w[0], w[1], w[2]}, {y[0], y[1], y[2]}, {n[0], n[1], n[2]}, {n[0], n[0] + n[1], N}};
            return launch_tile_mats(id, x, x_stride, mats, nullptr, 0, M, N, K, nullptr, s);
        }
    }
    int rc = launch_gemm_ws(x, x_stride, w[0], y[0], n[0], nullptr, 0, M, n[0], K, nullptr, ws, ws_bytes, s);
    if (rc) return rc;
    return launch_gemm_pair_ws(x, x_stride, w[1], y[1], n[1], w[2], y[2], n[2], M, K, ws, ws_bytes, s);
}

int launch_gemm_pair_ws(const uint16_t* x, int64_t x_stride, const uint16_t* w1, uint16_t* y1, int N1,
                        const uint16_t* w2, uint16_t* y2, int N2, int M, int K, void* ws, size_t ws_bytes,
                        hipStream_t s) {
    if (M == 0) return VITCOP_OK;
    const size_t need = gemm_skinny_workspace_bytes(M, N1 + N2, K);
    if (ws && need && ws_bytes >= need && N1 % 128 == 0 && N2 % 128 == 0)
        return launch_gemm_skinny(x, x_stride, w1, y1, N1, nullptr, 0, M, N1 + N2, K, nullptr, w2, y2, N1, ws, s);
    if (ws && ws_bytes >= splitk_workspace_bytes(M, N1 + N2, K) && N1 % 256 == 0 && N2 % 256 == 0) {
        const SplitKPlan p = splitk_plan(M, N1 + N2, K);              // (no tile of 256 columns straddles the two outputs)
        if (p.splits)
            return launch_gemm_splitk(p, x, x_stride, w1, y1, N1, nullptr, 0, M, N1 + N2, K, nullptr, ws, s, nullptr, 0.f,
                                      nullptr, 0, w2, y2, N1);
    }
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

size_t gemm_qkv_workspace_bytes(int M, int Hq, int Hkv, int d, int K) {
    const int qd = Hq * d, kd = Hkv * d;
    size_t need = std::max(gemm_workspace_bytes(M, kd, K), gemm_workspace_bytes(M, qd + kd, K));
    need = std::max(need, gemm_workspace_bytes(M, kd + qd + kd, K));
    // slices of the three together: what the next multiple of 64 rows takes, so that what a caller reserves up to some
    // number of rows grows with it (gemm_scratch_upto in api.hip); a launch takes as many slices as that holds
    const int R = (M + 63) / 64 * 64, path = qkv_path(R, qd, kd, d, K);
    if (path == 2) need = std::max(need, splitk_workspace_bytes(R, kd, K) + splitk_workspace_bytes(R, qd + kd, K));
    if (path == 3) need = std::max(need, up256((size_t)qkv_plan(R, qd, kd, K).splits * R * (qd + 2 * kd) * 4));
    return need;
}

int launch_gemm_qkv_rope_ws(const uint16_t* x, int64_t x_stride, const uint16_t* wk, const uint16_t* wq,
                            const uint16_t* wv, uint16_t* k_tmp, uint16_t* q, uint16_t* v_tmp, int Hq, int Hkv, int d,
                            const int32_t* positions, float theta, int M, int K, void* ws, size_t ws_bytes,
                            uint16_t* k_dst, uint16_t* v_dst, int T, int64_t kv_batch, hipStream_t s,
                            const int32_t* rows, SkParts* parts_out) {
    if (parts_out) parts_out->part = nullptr;
    if (M == 0) return VITCOP_OK;
    const int qd = Hq * d, kd = Hkv * d;
    const uint16_t* const w3[3] = {wk, wq, wv};
    // (rows that lie side by side: the projections write them where they belong, and k is turned in place)
    const bool dense = !rows && (M <= T || kv_batch == (int64_t)T * kd);
    uint16_t* const y3[3] = {dense ? k_dst : k_tmp, q, dense ? v_dst : v_tmp};
    const int n3[3] = {kd, qd, kd};
    const int path = ws ? qkv_path(M, qd, kd, d, K) : 0;
    QkvParts P{};
    if (path == 1 && ws_bytes >= gemm_skinny_workspace_bytes(M, kd + qd + kd, K)) {
        SkParts parts{};
        const int rc = launch_gemm_skinny3(x, x_stride, w3, y3, n3, M, K, ws, s, &parts);
        if (rc) return rc;
        if (parts_out && parts.part) {               // the caller finishes the rows itself
            *parts_out = parts;
            return VITCOP_OK;
        }
        // (no partial sums: the outputs are written already)
        P = {{parts, parts, parts}, {0, kd, kd + qd}};
    } else {
        const int N = qd + 2 * kd;
        SplitKPlan p;
        if (path == 3) p = qkv_plan(M, qd, kd, K, (int)std::min(ws_bytes / ((size_t)M * N * 4), (size_t)16));
        const size_t need_k = splitk_workspace_bytes(M, kd, K), need_qv = splitk_workspace_bytes(M, qd + kd, K);
        if (p.splits) {
            const SkParts parts{static_cast<float*>(ws), p.splits, N, M};
            const SkMats mats{{wk, wq, wv}, {y3[0], q, y3[2]}, {kd, qd, kd}, {kd, kd + qd, N}};
            const int rc = launch_slices(p, x, x_stride, mats, M, N, K, static_cast<float*>(ws), s);
            if (rc) return rc;
            P = {{parts, parts, parts}, {0, kd, kd + qd}};
        } else if (path == 2 && ws_bytes >= need_k + need_qv) {
            SkParts pk{}, pqv{};
            int rc = launch_gemm_splitk(splitk_plan(M, kd, K), x, x_stride, wk, y3[0], kd, nullptr, 0, M, kd, K, nullptr,
                                        ws, s, nullptr, 0.f, nullptr, 0, nullptr, nullptr, 0, &pk);
            if (rc) return rc;
            rc = launch_gemm_splitk(splitk_plan(M, qd + kd, K), x, x_stride, wq, q, qd, nullptr, 0, M, qd + kd, K, nullptr,
                                    static_cast<char*>(ws) + need_k, s, nullptr, 0.f, nullptr, 0, wv, y3[2], qd, &pqv);
            if (rc) return rc;
            P = {{pk, pqv, pqv}, {0, 0, qd}};
        } else {
            const int rc = launch_gemm_triple_ws(x, x_stride, w3, y3, n3, M, K, ws, ws_bytes, s);
            if (rc) return rc;
        }
    }
    if (P.parts[0].part != nullptr)
        return launch_qkv_finish(P, k_dst, q, v_dst, Hq, Hkv, d, positions, theta, T, kv_batch, s, rows);
    if (dense) return launch_rope(q, k_dst, positions, M, Hq, Hkv, d, theta, s);
    return launch_rope_append(q, k_tmp, v_tmp, positions, M, Hq, Hkv, d, theta, k_dst, v_dst, T, kv_batch, s, rows);
}

// Inner products between the rows of each of `batch` bf16 matrices f [n,K] (row stride and batch stride in elements), in
// fp32: gram[b][i][j] + gram[b][j][i] = <f_i, f_j> for i != j, sq[b][i] + (sq + sq_half)[b][i] = <f_i, f_i>.  The rows of
// gram must be writable up to the next multiple of 4 entries (gram_stride % 4 == 0).
int launch_gram(const uint16_t* f, int64_t row_stride, int64_t batch_stride, float* sq, int64_t sq_batch, int64_t sq_half, float* gram,
                int64_t gram_stride, int64_t gram_batch, int n, int K, int batch, hipStream_t s) {
    if (n == 0 || batch == 0) return VITCOP_OK;
    // A launch of one round takes its tiles' loads of their two operands, about 50 KB/us a CU in these launches: half of the
    // tiles are saved by symmetry and the others cut over k in two, onto the smaller tiles unless they need more rounds (8 x 288
    // tokens x 4096: all 25 tiles of 64 x 64, after a launch for the sums of squares, 6.5 + 19.3 us; in halves 16 for both;
    // 1 x 1856 x 3584: 225 tiles of 128 x 128 5.2 + 36.7, 240 halves 25.5).
    auto cost = [&](int t) {
        const long side = (n + t - 1) / t, wgs = side * (side + 1) * batch;
        return (wgs + 255) / 256 * t;
    };
#define VITCOP_GRAM(BT)                                                                                            \
    return launch_gemm_cfg<BT, BT, 2, 2, GM_EPI_GRAM>(f, row_stride, sk_mats(f, nullptr, 0, n), nullptr, 0, n, n, K, sq, \
                                                      s, row_stride, gram, gram_stride, batch, batch_stride, sq_batch, \
                                                      gram_batch, sq_half)
    if (cost(64) <= cost(128)) VITCOP_GRAM(64);
    VITCOP_GRAM(128);
#undef VITCOP_GRAM
}

}  // namespace vitcop
