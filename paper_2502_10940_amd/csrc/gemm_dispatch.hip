// gemm_dispatch.hip -- which bf16 MFMA kernel runs each GEMM
// C[M][N] = sum_k P(m, k) Q(n, k) of the layer, and the library's tuning
// options.
//
//  * PP (gemm_pp.hip): 256 x 256 tiles, two wave groups in ping-pong: the
//    least traffic and time per flop once its tiles fill the 256 CUs.
//  * MID (gemm_mid.hip): 128 x 128, 128 x 64 or 64 x 64 tiles, for outputs
//    that would leave most CUs without a 256 x 256 tile (token batches of a few
//    thousand, products of width r).
//  * SKINNY (gemm_skinny.hip): the forward products of at most 32 tokens.
//  * STREAM (gemm_stream.hip): BM x 128 tiles; operands without 16-byte aligned
//    rows.
// PP and MID need 16-byte aligned rows.  They and SKINNY sum over k in increasing
// order (as STREAM does with unaligned operands), so the choice among them never
// changes a bit of an unsplit product's result.
#include <atomic>

#include "internal.hpp"

namespace cola {

namespace {
// process-wide tuning options (cola_set_option)
std::atomic<int> g_force_stream{0};
std::atomic<int> g_wgrad_pair{1};
std::atomic<int> g_fuse_gate{1};
std::atomic<int> g_tile{0};

// Tile and modelled cost of a route.  Each round of up to 256 tiles costs
// steps * (step + load * x) + store * x microseconds, x the share of the CUs
// with a tile in it (all CUs busy share L2 and HBM), after `fixed` for the launch,
// the first loads and the last stores.  Fitted to MI355X timings of the products of
// the LLaMA shapes (60M to 7B) at 256 to 65536 tokens run by themselves over and
// over; the model is within about 15 % of them.  It has no term for bytes: products
// that are bound by memory take up to twice its time within a step, where their
// operands come from HBM (60M dZ 70 us against 35, the 350M group's dZ 140 against 77,
// Y of the both-sigma 350M layer 49 against 25), on every route alike.  E.g. T = 1024, K1 of a 1B projection (N = 512, K = 2048):
// 256 x 256 tiles 42 us (8 of them), 128 x 128 17, 128 x 64 13, 64 x 64 10;
// T = 4096 at 7B (N = 1024, K = 4096): 75, 36, 45, 55; T = 16384: 108, 138,
// 164, 210.  Weight gradients of one launch (r = 512, 2048 x 2048): at
// T = 1024 28, 12, 11, 12 us; at T = 32768, with the best split each and the
// reduction, 164, 181, 233, 353.
struct RouteCost {
    int bm, bn;
    double fixed, step, load, store;
    double wstep, wload;                // step and load with both operands m-contiguous (weight gradients)
};
constexpr RouteCost kCost[] = {
    {0, 0, 0, 0, 0, 0, 0, 0},                            // AUTO
    {256, 128, 0, 0, 0, 0, 0, 0},                        // STREAM (not modelled)
    {256, 256, 7.0, 1.09, 0.42, 5.0, 1.20, 0.55},        // PP
    {128, 128, 5.0, 0.36, 0.15, 4.0, 0.36, 0.26},        // MID
    {128, 64, 5.0, 0.26, 0.06, 1.0, 0.26, 0.12},
    {64, 64, 5.0, 0.15, 0.06, 0.7, 0.15, 0.15},
};
constexpr int kRoutes[] = {ROUTE_PP, ROUTE_MID_128x128, ROUTE_MID_128x64, ROUTE_MID_64x64};
}  // namespace

int set_option(int option, int value) {
    if (value < 0 || value > (option == OPT_TILE ? 4 : 1)) return -1;
    switch (option) {
        case OPT_TILE: g_tile.store(value); return 0;
        case OPT_STREAM_ONLY: g_force_stream.store(value); return 0;
        case OPT_WGRAD_PAIR: g_wgrad_pair.store(value); return 0;
        case OPT_FUSE_GATE: g_fuse_gate.store(value); return 0;
        default: return -1;
    }
}

int get_option(int option) {
    switch (option) {
        case OPT_STREAM_ONLY: return g_force_stream.load();
        case OPT_WGRAD_PAIR: return g_wgrad_pair.load();
        case OPT_FUSE_GATE: return g_fuse_gate.load();
        case OPT_TILE: return g_tile.load();
        default: return -1;
    }
}

int64_t route_tiles(int route, int64_t M, int64_t N) {
    const RouteCost& c = kCost[route];
    return ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
}

double route_us(int route, int64_t tiles, int64_t steps, bool wgrad) {
    const RouteCost& c = kCost[route];
    const double full = (double)(tiles / 256);
    const double x = (double)(tiles % 256) / 256.0;            // the last round's share of the CUs
    const double step = wgrad ? c.wstep : c.step, load = wgrad ? c.wload : c.load;
    return c.fixed + full * ((double)steps * (step + load) + c.store) +
           (x > 0.0 ? (double)steps * (step + load * x) + c.store * x : 0.0);
}

bool route_fits(int route, int64_t M, int64_t N, int64_t splits) {
    if (route == ROUTE_PP) return M >= 128 && N >= 128;
    return route_tiles(route, M, N) * splits < kMidMaxBlocks;
}

int asked_route() {
    const int t = g_tile.load(std::memory_order_relaxed);
    return t ? ROUTE_PP + t - 1 : ROUTE_AUTO;
}

int gemm_route(int64_t M, int64_t N, int64_t K) {
    if (g_force_stream.load(std::memory_order_relaxed)) return ROUTE_STREAM;
    if (asked_route() != ROUTE_AUTO && route_fits(asked_route(), M, N, 1)) return asked_route();
    const int64_t steps = (K + BF16_BK - 1) / BF16_BK;
    int best = ROUTE_STREAM;
    double best_us = -1.0;
    for (int r : kRoutes) {
        if (!route_fits(r, M, N, 1)) continue;
        const int64_t tiles = route_tiles(r, M, N);
        double us = route_us(r, tiles, steps, false);
        // 256 x 256 tiles on half the CUs or more give way only to a gain above the
        // model's error: the CUs they leave free are not lost to a caller with a
        // second stream, and work per CU is the better.  Z and dZ of the 350M shape
        // at 32768 tokens (128 such tiles), two streams: a step of 7 projections
        // takes 1.51 ms with them and 1.69 with the 128 x 128 tiles that the model
        // prefers by 3 to 13 %; one stream 2.17 and 2.15.  Not with a short K, where
        // a tile is mostly its stores (dX of 8192 x 1024, K = 256: the both-sigma
        // layer's step 167.5 us with 128 x 64 tiles, 169.0 with 256 x 256).
        if (r == ROUTE_PP && tiles >= 128 && steps >= 8) us *= 0.85;
        if (best_us < 0 || us < best_us) {
            best_us = us;
            best = r;
        }
    }
    return best;
}

// PP and MID take only operands with 16-byte aligned rows whose tile offsets
// fit their 32-bit per-lane offsets.
static bool operands_ok(const GemmArgs& a) {
    auto al = [](const void* p, int64_t ld) {
        return (reinterpret_cast<uintptr_t>(p) & 15u) == 0 && (ld & 7) == 0 && ld < (int64_t(1) << 22);
    };
    return al(a.p, a.ldp) && al(a.q, a.ldq);
}

// Up to 32 tokens: one token of a 1B projection 9.4 us of kernels against 14.3
// with 64 x 64 tiles, 32 tokens of 7B q, k, v 18.6 against 34.  With a 64-row variant
// of the kernel, 48 tokens of a 1B projection took 14.2 us against 13.5 with MID
// tiles, of 7B 20.9 against 20.1, of 7B gate and up 32.9 against 24.8.
bool skinny_rows(int64_t M) {
    return M <= kSkinnyRows && !g_force_stream.load(std::memory_order_relaxed) && asked_route() == ROUTE_AUTO;
}

static bool skinny_takes(const GemmArgs& a) {
    return skinny_rows(a.M) && a.splits == 1 && a.p_layout == KMAJ && a.q_layout == KMAJ &&
           (a.tag == TAG_FWD_Z || a.tag == TAG_INFER_H || a.tag == TAG_FWD_Y || a.tag == TAG_FWD_YP);
}

static int route_of(const GemmArgs& a) {
    if (skinny_takes(a)) return ROUTE_SKINNY;
    if (!operands_ok(a)) return ROUTE_STREAM;
    return a.route != ROUTE_AUTO ? a.route : gemm_route(a.M, a.N, a.K);
}

static hipError_t launch_route(const GemmArgs* a, int n, int route, hipStream_t s) {
    if (route >= ROUTE_MID_128x128) {
        for (int i = 0; i < n; i += kMidBatch) {
            const int m = n - i < kMidBatch ? n - i : kMidBatch;
            const hipError_t e = route == ROUTE_SKINNY ? launch_gemm_skinny(a + i, m, s)
                                                       : launch_gemm_mid(a + i, m, route - ROUTE_MID_128x128, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    for (int i = 0; i < n; ++i) {
        const hipError_t e = route == ROUTE_PP ? launch_gemm_pp(a[i], s) : launch_gemm_stream(a[i], s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

bool fused_epilogue_takes(const GemmArgs& a) { return route_of(a) != ROUTE_STREAM; }

hipError_t launch_gemm_bf16_wgrads(const GemmArgs* a, int n, hipStream_t s) {
    bool alike = n <= kMidBatch;
    for (int i = 0; i < n; ++i) alike = alike && route_of(a[i]) == route_of(a[0]);
    if (alike && route_of(a[0]) == ROUTE_PP) return launch_gemm_pp_batch(a, n, s);
    if (alike) return launch_route(a, n, route_of(a[0]), s);
    for (int i = 0; i < n; ++i) {
        const hipError_t e = launch_gemm_bf16(a[i], s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// While all tiles of the weight gradients' route run at once (two workgroups a
// CU): a launch less, and either part fills the CUs the other leaves idle.
bool bf16_dxw_takes(const GemmArgs* a, int n) {
    if (n > kMidBatch || (a[1].route != ROUTE_MID_128x64 && a[1].route != ROUTE_MID_64x64)) return false;
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) {
        if (!operands_ok(a[i]) || (i > 0 && a[i].route != a[1].route)) return false;
        tiles += route_tiles(a[1].route, a[i].M, a[i].N) * a[i].splits;
    }
    return tiles <= 512 && !g_force_stream.load(std::memory_order_relaxed);
}

hipError_t launch_gemm_bf16_dxw(const GemmArgs* a, int n, hipStream_t s) {
    return launch_gemm_mid_dxw(a, n, a[1].route - ROUTE_MID_128x128, s);
}

hipError_t launch_gemm_bf16_batch(const GemmArgs* a, int n, hipStream_t s) {
    int64_t K = 0;
    bool skinny = n > 1, ok = n > 1 && n <= kMidBatch && !g_force_stream.load(std::memory_order_relaxed);
    for (int i = 0; i < n; ++i) {
        skinny = skinny && skinny_takes(a[i]) && a[i].epi == a[0].epi;
        ok = ok && operands_ok(a[i]) && a[i].splits == 1 && a[i].epi == a[0].epi;
        K = a[i].K > K ? a[i].K : K;
    }
    if (skinny) return launch_route(a, n, ROUTE_SKINNY, s);
    if (ok) {
        // Together on one route (their tiles run at once: four dZ products of 64
        // 256 x 256 tiles fill the CUs that one leaves three quarters idle) or
        // one by one, whichever the model says is faster.  256 x 256 tiles share a
        // launch only while they fit one round: beyond it the persistent kernel
        // of each product alone is the faster (2 x 1408 tiles with K = 256: 174
        // us against 184 together; 2 x 128 tiles with K = 2736: 216 against 140).
        const int64_t steps = (K + BF16_BK - 1) / BF16_BK;
        int best = ROUTE_AUTO;
        double best_us = 0.0;
        for (int i = 0; i < n; ++i) {
            const int r = gemm_route(a[i].M, a[i].N, a[i].K);
            best_us += r == ROUTE_STREAM ? 1e30 : route_us(r, route_tiles(r, a[i].M, a[i].N), steps, false);
        }
        for (int r : kRoutes) {
            int64_t tiles = 0;
            bool fits = r != ROUTE_PP || a[0].epi == EPI_DZ || (a[0].epi == EPI_STORE && a[0].q_layout == KMAJ);
            for (int i = 0; i < n; ++i) {
                tiles += route_tiles(r, a[i].M, a[i].N);
                fits = fits && route_fits(r, a[i].M, a[i].N, n);
            }
            fits = fits && (r != ROUTE_PP || tiles <= 256);
            const double us = route_us(r, tiles, steps, false);
            if (fits && (us < best_us || r == asked_route())) {
                best_us = us;
                best = r;
                if (r == asked_route()) break;
            }
        }
        if (asked_route() != ROUTE_AUTO && best != asked_route()) best = ROUTE_AUTO;
        if (best == ROUTE_PP) return launch_gemm_pp_batch(a, n, s);
        if (best != ROUTE_AUTO) return launch_route(a, n, best, s);
    }
    for (int i = 0; i < n; ++i) {
        const hipError_t e = launch_gemm_bf16(a[i], s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_gemm_bf16(const GemmArgs& a, hipStream_t s) { return launch_route(&a, 1, route_of(a), s); }

}  // namespace cola
