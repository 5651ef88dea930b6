// cola_abi.hip -- the C ABI of libcola.so (include/cola.h): argument
// validation, workspace planning, the launch sequence of each call, and the
// optional per-kernel event timing.
//
// Launch sequences (one stream, no host synchronisation):
//   cola_fwd : K1  Z = X A^T, H = sigma(Z)          (epilogue writes Z and H)
//              K2  Y = H B^T
//   cola_bwd : K3  dZ = (dY B) (.) sigma'(Z)        (CoLA-M: also H = sigma(Z))
//              K4  dX = dZ A
//              K5  dA partials = dZ^T X             (split over tokens)
//              K6  dB partials = dY^T H             (split over tokens)
//                  (K5 and K6 in one launch, one split of T for both)
//              K7  dA, dB = fixed-order sums of the partials
//                  (small layers: K4, K5 and K6 in one launch)
//   dense    : Y = X W^T ; dX = dY W ; dW = dY^T X (split over tokens + K7)
#include <mutex>
#include <new>
#include <stdio.h>
#include <string.h>
#include <vector>

#include "../../include/cola.h"
#include "internal.hpp"
#include "block.hpp"

using namespace cola;

namespace {

thread_local char g_err[256] = "";

int hip_fail(hipError_t e, const char* where) {
    snprintf(g_err, sizeof(g_err), "%s: %s", where, hipGetErrorString(e));
    return COLA_ERR_HIP;
}

// ---------------------------------------------------------------------------
// timing
// ---------------------------------------------------------------------------
struct Timed {
    hipEvent_t start, stop;
    int kc;
    double flops, bytes;
};

struct TimingState {
    std::mutex mu;
    bool on = false;
    std::vector<Timed> pending;
    std::vector<hipEvent_t> free_events;
    int64_t launches[COLA_KC_COUNT] = {};
    double ms[COLA_KC_COUNT] = {};
    double flops[COLA_KC_COUNT] = {};
    double bytes[COLA_KC_COUNT] = {};
};

TimingState& timing() {
    static TimingState* t = new TimingState();   // never destroyed: events may outlive static dtors
    return *t;
}

hipError_t get_event(TimingState& t, hipEvent_t* e) {
    if (!t.free_events.empty()) {
        *e = t.free_events.back();
        t.free_events.pop_back();
        return hipSuccess;
    }
    return hipEventCreate(e);
}

// Drain recorded events into the totals (waits for them).
hipError_t drain(TimingState& t) {
    for (const Timed& x : t.pending) {
        hipError_t e = hipEventSynchronize(x.stop);
        if (e != hipSuccess) return e;
        float ms = 0.f;
        e = hipEventElapsedTime(&ms, x.start, x.stop);
        if (e != hipSuccess) return e;
        t.launches[x.kc] += 1;
        t.ms[x.kc] += ms;
        t.flops[x.kc] += x.flops;
        t.bytes[x.kc] += x.bytes;
        t.free_events.push_back(x.start);
        t.free_events.push_back(x.stop);
    }
    t.pending.clear();
    return hipSuccess;
}

// Run one launch, bracketed by events when timing is on.
template <class F>
hipError_t timed(int kc, double flops, double bytes, hipStream_t s, F&& launch) {
    TimingState& t = timing();
    if (!t.on) return launch();
    std::lock_guard<std::mutex> lock(t.mu);
    if (t.pending.size() >= 8192) {
        hipError_t e = drain(t);
        if (e != hipSuccess) return e;
    }
    Timed x{};
    x.kc = kc; x.flops = flops; x.bytes = bytes;
    hipError_t e = get_event(t, &x.start);
    if (e == hipSuccess) e = get_event(t, &x.stop);
    if (e == hipSuccess) e = hipEventRecord(x.start, s);
    if (e != hipSuccess) return e;
    e = launch();
    if (e != hipSuccess) return e;
    e = hipEventRecord(x.stop, s);
    if (e != hipSuccess) return e;
    t.pending.push_back(x);
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// shapes and plans
// ---------------------------------------------------------------------------
constexpr int64_t kMaxDim = int64_t(1) << 40;   // keeps every byte count far from overflow
static_assert(COLA_MAX_PITCH == kMaxPitch, "the public pitch limit is the kernels' limit");

struct Dims {
    int64_t T, d_in, d_out, r, ldx, ldy, ldz;
    bool bf16;
    size_t esize;
};

bool valid_act(int act) { return act == COLA_ACT_IDENTITY || act == COLA_ACT_SILU || act == COLA_ACT_GELU; }

int check_desc(const cola_desc* d, Dims* out) {
    if (!d) return COLA_ERR_INVALID_ARG;
    if (d->dtype != COLA_F32 && d->dtype != COLA_BF16) return COLA_ERR_INVALID_ARG;
    if (!valid_act(d->act)) return COLA_ERR_INVALID_ARG;
    if (d->recompute != 0 && d->recompute != 1) return COLA_ERR_INVALID_ARG;
    if (d->T < 0 || d->d_in < 1 || d->d_out < 1 || d->r < 1) return COLA_ERR_BAD_SHAPE;
    if (d->T > kMaxDim || d->d_in > kMaxDim || d->d_out > kMaxDim || d->r > kMaxDim)
        return COLA_ERR_BAD_SHAPE;
    Dims x;
    x.T = d->T; x.d_in = d->d_in; x.d_out = d->d_out; x.r = d->r;
    x.ldx = d->ldx ? d->ldx : d->d_in;
    x.ldy = d->ldy ? d->ldy : d->d_out;
    x.ldz = d->ldz ? d->ldz : d->r;
    if (x.ldx < x.d_in || x.ldy < x.d_out || x.ldz < x.r) return COLA_ERR_BAD_SHAPE;
    if (x.ldx > kMaxPitch || x.ldy > kMaxPitch || x.ldz > kMaxPitch) return COLA_ERR_BAD_SHAPE;
    // element counts of the largest operands must stay below 2^62
    const double big = (double)x.T * (double)(x.ldx > x.ldy ? x.ldx : x.ldy);
    if (big > 4.0e18 || (double)x.r * (double)(x.d_in > x.d_out ? x.d_in : x.d_out) > 4.0e18)
        return COLA_ERR_BAD_SHAPE;
    x.bf16 = d->dtype == COLA_BF16;
    x.esize = x.bf16 ? 2 : 4;
    *out = x;
    return COLA_OK;
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Split of a token-long (K = T) weight-gradient GEMM into chunks of whole K
// tiles, and the kernel it was planned for.  Depends only on the shape (and
// the tuning options), so results are reproducible run to run; in particular not
// on the room for copies of unaligned rows, nor on whether H is stored: the kernels
// for aligned and for unaligned rows sum a chunk in the same order, so that dA and
// dB have the same bits in every workspace, in CoLA and in CoLA-M.
struct Split {
    int splits;
    int64_t k_chunk;
    int route;
};

struct WShape {
    int64_t M, N;
};

constexpr int64_t kMaxSplits = 64;

// Bytes of the fp32 partials of n products (none for one split).
size_t partial_bytes(const WShape* w, int n, int64_t splits) {
    size_t b = 0;
    for (int i = 0; i < n && splits > 1; ++i) b += align256((size_t)splits * (size_t)(w[i].M * w[i].N) * 4);
    return b;
}

// Tiles of the streaming family: 256 x 128, or 128 x 128 for at most 128 rows.
int64_t stream_tiles(const WShape& w) {
    const int64_t bm = w.M > 128 ? 256 : 128;
    return ((w.M + bm - 1) / bm) * ((w.N + 127) / 128);
}

// Split of the streaming family: the split count S minimises rounds(S) * ceil(ktiles / S) K-tile steps of about 2 us
// each, where rounds(S) = ceil(tiles * S / slots) and slots is the number of
// workgroups the chip runs at once -- a split that leaves a few workgroups for a
// second round costs a whole round -- plus writing and re-reading the S fp32
// partials (`elems` values per split) at about 4 TB/s.
Split plan_split_tiles(int64_t bk, int64_t tiles, int64_t slots, int64_t K, double elems) {
    const int64_t ktiles = (K + bk - 1) / bk;
    if (ktiles < 1) return Split{1, bk, ROUTE_AUTO};           // empty batch: nothing to split
    const double step_us = 2.0;
    const double partial_us_per_split = elems * 8.0 / 4.0e6;
    int64_t maxs = ktiles / 4;
    if (maxs < 1) maxs = 1;
    if (maxs > kMaxSplits) maxs = kMaxSplits;
    int64_t best_s = 1;
    double best_cost = -1.0;
    for (int64_t s = 1; s <= maxs; ++s) {
        const int64_t chunk = (ktiles + s - 1) / s;
        const int64_t eff_s = (ktiles + chunk - 1) / chunk;   // splits actually used
        const int64_t rounds = (tiles * eff_s + slots - 1) / slots;
        const double cost = (double)(rounds * chunk) * step_us +
                            (eff_s > 1 ? (double)eff_s * partial_us_per_split : 0.0);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best_s = s;
        }
    }
    const int64_t chunk_tiles = (ktiles + best_s - 1) / best_s;
    Split s;
    s.k_chunk = chunk_tiles * bk;
    s.splits = (int)((K + s.k_chunk - 1) / s.k_chunk);
    if (s.splits < 1) s.splits = 1;
    s.route = ROUTE_AUTO;
    return s;
}

// Route and split of the n weight gradients that share a launch and one split
// of K = T: the pair that minimises the routes' cost model (which covers storing
// the partials) plus the reduction: its launch (2 us), and the partials and the
// result at about 5 TB/s (8 splits of 2.1 M values: 14 us; 2 of 8.4 M: 18 us).
// `stream`: planned for the streaming family.  `room`: for the partials.
Split plan_split_bf16(const WShape* w, int n, int64_t K, bool stream, size_t room) {
    const int64_t ktiles = (K + BF16_BK - 1) / BF16_BK;
    if (ktiles < 1) return Split{1, BF16_BK, ROUTE_AUTO};
    double elems = 0.0;
    for (int i = 0; i < n; ++i) elems += (double)w[i].M * (double)w[i].N;
    if (stream || get_option(OPT_STREAM_ONLY) == 1) {
        int64_t tiles = 0;
        for (int i = 0; i < n; ++i) tiles += stream_tiles(w[i]);
        return plan_split_tiles(BF16_BK, tiles, 512, K, elems);
    }
    int64_t maxs = ktiles / 4;
    if (maxs < 1) maxs = 1;
    if (maxs > kMaxSplits) maxs = kMaxSplits;
    Split best{1, ktiles * BF16_BK, ROUTE_AUTO};
    double best_cost = -1.0;
    for (int route = ROUTE_PP; route <= ROUTE_MID_64x64; ++route) {
        int64_t tiles = 0;
        bool fits = true;
        for (int i = 0; i < n; ++i) {
            tiles += route_tiles(route, w[i].M, w[i].N);
            fits = fits && route_fits(route, w[i].M, w[i].N, maxs);
        }
        if (!fits) continue;
        if (route == asked_route()) best_cost = -1.0;          // whatever the others cost
        for (int64_t s = 1; s <= maxs; ++s) {
            const int64_t chunk = (ktiles + s - 1) / s;
            const int64_t eff_s = (ktiles + chunk - 1) / chunk;
            if (partial_bytes(w, n, eff_s) > room) break;
            const double cost = route_us(route, tiles * eff_s, chunk, true) +
                                (eff_s > 1 ? 2.0 + (double)(eff_s + 1) * elems * 4.0 / 5.0e6 : 0.0);
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                best = Split{(int)eff_s, chunk * BF16_BK, route};
            }
        }
        if (route == asked_route()) break;
    }
    return best;
}

// Split of the fp32 weight gradients that share a launch: a workgroup of 32 x 32
// tiles takes eight K tiles at once in about 0.9 us (a CU's matrix cores need that
// long for them), against the reduction's launch (4 us) and partials at about
// 4 TB/s.
Split plan_split_f32(const WShape* w, int n, int64_t K, size_t room) {
    const int64_t steps = (K + 8 * F32_BK - 1) / (8 * F32_BK);
    if (steps < 1) return Split{1, F32_BK, ROUTE_AUTO};
    double elems = 0.0;
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) {
        elems += (double)w[i].M * (double)w[i].N;
        tiles += f32_tiles(32, w[i].M, w[i].N);
    }
    Split best{1, steps * 8 * F32_BK, ROUTE_AUTO};
    double best_cost = -1.0;
    for (int64_t s = 1; s <= (steps < kMaxSplits ? steps : kMaxSplits); ++s) {
        const int64_t chunk = (steps + s - 1) / s;
        const int64_t eff_s = (steps + chunk - 1) / chunk;
        if (partial_bytes(w, n, eff_s) > room) break;
        const double rounds = (double)((tiles * eff_s + 255) / 256);
        const double cost = rounds * (double)chunk * 0.9 + (eff_s > 1 ? 4.0 + (double)eff_s * elems * 8.0 / 4.0e6 : 0.0);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = Split{(int)eff_s, chunk * 8 * F32_BK, ROUTE_AUTO};
        }
    }
    return best;
}

Split plan_split(bool bf16, const WShape* w, int n, int64_t K, bool stream = false, size_t room = SIZE_MAX) {
    return bf16 ? plan_split_bf16(w, n, K, stream, room) : plan_split_f32(w, n, K, room);
}

// The two weight gradients of a layer in one launch: their tiles share the slots
// and one split of K = T.  The option COLA_OPT_WGRAD_PAIR = 0 launches them one by
// one (tuning, comparisons).
bool pair_wgrads(bool bf16) {
    return get_option(OPT_WGRAD_PAIR) == 1 && (!bf16 || get_option(OPT_STREAM_ONLY) == 0);
}

// Room for the partials of a layer's weight gradients that share a launch (n = 2)
// or do not (n = 1): what the splits of the 256 x 256, streaming and 64 x 64 fp32
// kernels take.  A rule of its own, so that the calls that cola_bwd_scratch accepts
// do not move with the choice of kernels, and that call and cola_bwd have one plan.
// It binds in 2 of 3000 shapes of 16 to 65536 tokens, 64 to 11008 wide: the others'
// splits for smaller tiles take less.
size_t partial_room(bool bf16, const WShape* w, int n, int64_t T) {
    const bool stream = get_option(OPT_STREAM_ONLY) == 1;
    const int64_t bk = bf16 ? 64 : 16;
    int64_t tiles[2] = {0, 0}, slots[2] = {0, 0};
    bool wide = n == 2;
    for (int i = 0; i < n; ++i) {
        const bool pp = bf16 && !stream && w[i].M >= 128 && w[i].N >= 128;
        wide = wide && pp;
        tiles[i] = !bf16 ? f32_tiles(64, w[i].M, w[i].N) : (pp ? f32_tiles(256, w[i].M, w[i].N) : stream_tiles(w[i]));
        slots[i] = !bf16 ? 1024 : (pp ? 256 : 512);
    }
    auto elems = [&](int i) { return (double)w[i].M * (double)w[i].N; };
    if (wide)
        return partial_bytes(w, 2, plan_split_tiles(bk, tiles[0] + tiles[1], 256, T, elems(0) + elems(1)).splits);
    size_t b = 0;
    for (int i = 0; i < n; ++i) b += partial_bytes(w + i, 1, plan_split_tiles(bk, tiles[i], slots[i], T, elems(i)).splits);
    return b;
}

// Rows of pitch ld start on 16-byte boundaries (bf16).
bool pitch16(int64_t ld) { return ld % 8 == 0; }

// Row pitch (elements) of a buffer the library lays out itself: a whole
// number of 128-byte cache lines, so every K tile of a row starts on a line
// (rows that straddle lines cost up to 1.4x on MI355X, measured).
int64_t line_pitch(bool bf16, int64_t width) {
    const int64_t per = bf16 ? 64 : 32;
    return (width + per - 1) / per * per;
}

// A bf16 operand whose rows are not a whole number of 16-byte chunks apart is
// copied to the workspace with a line-aligned pitch, so that the fast MFMA
// kernels, whose loads need aligned rows, take the products that read it.
// Weights (contiguous rows, width not a multiple of 8) and token rows (pitch
// not a multiple of 8).  One pass over the operand instead of element loads in
// every product: X A^T of 4095 tight rows of 5461 took 960 us with them, 36 us
// and a 20 us copy without (MI355X).  Depends only on the shape.
struct Pack {
    bool on;
    int64_t rows, width;
    int64_t ld;     // pitch to use for the operand
    size_t off, bytes;
};

Pack plan_pack(bool on, int64_t rows, int64_t width, int64_t ld, size_t off) {
    Pack p;
    p.off = off;
    p.on = on;
    p.rows = rows;
    p.width = width;
    p.ld = p.on ? line_pitch(true, width) : ld;
    p.bytes = p.on ? align256((size_t)rows * (size_t)p.ld * 2) : 0;
    return p;
}

Pack plan_weight(bool bf16, int64_t rows, int64_t width, size_t off) {
    return plan_pack(bf16 && !pitch16(width), rows, width, width, off);
}

// The forward products of a few tokens take rows of any alignment: a copy of
// operands that are read once would only add a pass.
Pack direct(Pack p, bool skinny, int64_t src_ld) {
    if (skinny && p.on) {
        p.on = false;
        p.ld = src_ld;
    }
    return p;
}

// Resolve an operand (rows src_ld apart) to a pointer, enqueueing its copy if
// planned; its pitch is pk.ld.
hipError_t use_packed(const Pack& pk, const void* src, int64_t src_ld, char* ws, const void** out, hipStream_t s) {
    if (!pk.on) {
        *out = src;
        return hipSuccess;
    }
    *out = ws + pk.off;
    return launch_pack_rows(src, src_ld, pk.rows, pk.width, ws + pk.off, pk.ld, s);
}

// Token rows are copied when the workspace has room for them (`copies`: a mask); a
// caller that brings only the `lean` size gets the kernels for unaligned rows (the
// same bits, more slowly).
// cola_workspace_bytes returns the full size.
enum Copies : unsigned { COPY_DY = 1, COPY_H = 2, COPY_X = 4 };
constexpr unsigned kAllCopies = COPY_DY | COPY_H | COPY_X;

// The copies that a queried size has room for; takes COLA_WS_LEAN off the phase.
unsigned phase_copies(int* phase) {
    const bool lean = *phase >= COLA_WS_LEAN;
    if (lean) *phase -= COLA_WS_LEAN;
    return lean ? 0 : kAllCopies;
}

struct FwdPlan {
    int64_t ldw;          // pitch of the workspace copy of H (CoLA-M)
    size_t off_h, total;
    Pack pa, pb;          // repacked A [r][d_in] and B [d_out][r]
    Pack px, ph;          // repacked X and H
};

FwdPlan plan_fwd(const Dims& x, bool recompute, unsigned copies = kAllCopies) {
    FwdPlan p;
    p.ldw = line_pitch(x.bf16, x.r);
    p.off_h = 0;
    const size_t hbytes = recompute ? align256((size_t)x.T * (size_t)p.ldw * x.esize) : 0;
    p.pa = plan_weight(x.bf16, x.r, x.d_in, hbytes);
    p.pb = plan_weight(x.bf16, x.d_out, x.r, p.pa.off + p.pa.bytes);
    if (!x.bf16) copies = 0;
    p.px = plan_pack((copies & COPY_X) && !pitch16(x.ldx), x.T, x.d_in, x.ldx, p.pb.off + p.pb.bytes);
    p.ph = plan_pack((copies & COPY_H) && !recompute && !pitch16(x.ldz), x.T, x.r, recompute ? p.ldw : x.ldz,
                     p.px.off + p.px.bytes);
    p.total = p.ph.off + p.ph.bytes;
    if (x.T == 0) p.total = 0;
    return p;
}

struct BwdPlan {
    int64_t ldw;          // pitch of dZ (and recomputed H) in the workspace
    size_t off_dz, off_h, off_pa, off_pb, total;
    Split sa, sb;         // the same split for both when pair
    bool pair;            // dA and dB in one launch
    Pack wa, wb;          // repacked A and B
    Pack px, py, ph;      // repacked X, dY and H
};

BwdPlan plan_bwd(const Dims& x, bool recompute, unsigned copies = kAllCopies) {
    BwdPlan p;
    p.ldw = line_pitch(x.bf16, x.r);
    const size_t zbytes = align256((size_t)x.T * (size_t)p.ldw * x.esize);
    if (!x.bf16) copies = 0;
    p.pair = pair_wgrads(x.bf16);
    const WShape w[2] = {{x.r, x.d_in}, {x.d_out, x.r}};
    if (p.pair) {
        p.sa = p.sb = plan_split(x.bf16, w, 2, x.T, false, partial_room(x.bf16, w, 2, x.T));
    } else {
        p.sa = plan_split(x.bf16, w, 1, x.T, false, partial_room(x.bf16, w, 1, x.T));
        p.sb = plan_split(x.bf16, w + 1, 1, x.T, false, partial_room(x.bf16, w + 1, 1, x.T));
    }
    p.off_dz = 0;
    p.off_h = zbytes;
    p.off_pa = p.off_h + (recompute ? zbytes : 0);
    p.off_pb = p.off_pa + partial_bytes(w, 1, p.sa.splits);
    p.wa = plan_weight(x.bf16, x.r, x.d_in, p.off_pb + partial_bytes(w + 1, 1, p.sb.splits));
    p.wb = plan_weight(x.bf16, x.d_out, x.r, p.wa.off + p.wa.bytes);
    p.px = plan_pack((copies & COPY_X) && !pitch16(x.ldx), x.T, x.d_in, x.ldx, p.wb.off + p.wb.bytes);
    p.py = plan_pack((copies & COPY_DY) && !pitch16(x.ldy), x.T, x.d_out, x.ldy, p.px.off + p.px.bytes);
    p.ph = plan_pack((copies & COPY_H) && !recompute && !pitch16(x.ldz), x.T, x.r, recompute ? p.ldw : x.ldz,
                     p.py.off + p.py.bytes);
    p.total = p.ph.off + p.ph.bytes;
    if (x.T == 0) p.total = 0;
    return p;
}

// The plan that `ws_bytes` has room for: with every copy of unaligned rows, or with
// those that fit (dY first: two products read it, the dB of an uncopied H still one),
// or the lean one, which is refused if that is too large as well.  40000 tokens,
// 257 -> 255, r = 129 in cola_bwd_scratch: 826 us without copies, 429 with those of
// dY and H.
template <class F>
auto fitting(size_t ws_bytes, F&& plan) {
    auto p = plan(kAllCopies);
    constexpr unsigned order[] = {COPY_DY | COPY_H, COPY_DY | COPY_X, COPY_DY, COPY_H | COPY_X, COPY_X, 0u};
    for (unsigned copies : order) {
        if (ws_bytes >= p.total) break;
        p = plan(copies);
    }
    return p;
}

hipError_t gemm(const GemmArgs& a, bool bf16, hipStream_t s) {
    return bf16 ? launch_gemm_bf16(a, s) : launch_gemm_f32_batch(&a, 1, s);
}

// n products of one kind and step, timed as one launch of class kc.
hipError_t gemms(const GemmArgs* a, int n, int kc, double flops, double bytes, bool bf16, hipStream_t s) {
    if (n == 0) return hipSuccess;
    return timed(kc, flops, bytes, s, [&]() -> hipError_t {
        if (bf16) return launch_gemm_bf16_batch(a, n, s);
        for (int i = 0; i < n; i += kF32Batch) {
            const hipError_t e = launch_gemm_f32_batch(a + i, n - i < kF32Batch ? n - i : kF32Batch, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    });
}

GemmArgs make_args(int tag, int64_t M, int64_t N, int64_t K, const void* p, int64_t ldp, int pl,
                   const void* q, int64_t ldq, int ql, void* c, int64_t ldc, int epi, int act) {
    GemmArgs a{};
    a.tag = tag;
    a.M = M; a.N = N; a.K = K;
    a.p = p; a.ldp = ldp; a.p_layout = pl;
    a.q = q; a.ldq = ldq; a.q_layout = ql;
    a.c = c; a.ldc = ldc;
    a.epi = epi; a.act = act;
    a.splits = 1;
    a.k_chunk = K > 0 ? K : 1;
    a.split_stride = 0;
    return a;
}

double gemm_flops(int64_t M, int64_t N, int64_t K) { return 2.0 * (double)M * (double)N * (double)K; }

// A weight gradient C[M][N] = sum_t P[t][m] Q[t][n]; its partials, if split.
struct WProd {
    int64_t M, N;
    const void *P, *Q;
    int64_t ldp, ldq;
    float *C, *part;
    int kc;               // timing class on its own
};

// n weight gradients (n <= kWSet) over K = T in one launch with one split, then
// the fixed-order reductions of their partials in another.  `dx`: the dX = dZ A
// product not yet launched; it joins the launch where that is faster, or goes
// first in one of its own (bytes: its own traffic).
constexpr int kWSet = 4;
static_assert(kWSet <= kMidBatch && kWSet <= kF32Batch && kWSet <= kReduceBatch, "a set is one launch");

struct DxProd {
    GemmArgs a;
    double bytes;
};

int launch_dx(bool bf16, const DxProd& dx, hipStream_t s) {
    const hipError_t e = timed(COLA_KC_BWD_DX, gemm_flops(dx.a.M, dx.a.N, dx.a.K), dx.bytes, s,
                               [&] { return gemm(dx.a, bf16, s); });
    return e == hipSuccess ? COLA_OK : hip_fail(e, "bwd_dx");
}

int wgrads(bool bf16, int64_t T, const Split& sp, const WProd* w, int n, hipStream_t s, const DxProd* dx = nullptr) {
    GemmArgs all[kWSet + 1];
    GemmArgs* const a = all + 1;
    ReduceJob red[kWSet];
    double flops = 0.0, elems = 0.0, in = 0.0;
    for (int i = 0; i < n; ++i) {
        a[i] = make_args(i == 0 ? TAG_BWD_DA : TAG_BWD_DB, w[i].M, w[i].N, T, w[i].P, w[i].ldp, MNMAJ, w[i].Q, w[i].ldq,
                         MNMAJ, w[i].C, w[i].N, EPI_STORE_F32, 0);
        if (n == 1) a[i].tag = w[i].kc;
        a[i].splits = sp.splits;
        a[i].k_chunk = sp.k_chunk;
        a[i].route = sp.route;
        if (sp.splits > 1) {
            a[i].c = w[i].part;
            a[i].split_stride = w[i].M * w[i].N;
        }
        red[i] = ReduceJob{w[i].part, w[i].C, w[i].M * w[i].N};
        flops += gemm_flops(w[i].M, w[i].N, T);
        elems += (double)w[i].M * (double)w[i].N;
        in += (bf16 ? 2.0 : 4.0) * (double)T * (double)(w[i].M + w[i].N);
    }
    bool joined = false;
    if (dx) {
        all[0] = dx->a;
        joined = get_option(OPT_WGRAD_PAIR) == 1 &&
                 (bf16 ? bf16_dxw_takes(all, n + 1) : f32_dxw_takes(all, n + 1));
        if (!joined) {
            const int st = launch_dx(bf16, *dx, s);
            if (st != COLA_OK) return st;
        } else {
            flops += gemm_flops(dx->a.M, dx->a.N, dx->a.K);
            in += dx->bytes;
        }
    }
    const int kc = n > 1 || joined ? (int)COLA_KC_BWD_DADB : w[0].kc;
    hipError_t e = timed(kc, flops, in + elems * 4.0 * sp.splits, s, [&] {
        if (joined) return bf16 ? launch_gemm_bf16_dxw(all, n + 1, s) : launch_gemm_f32_dxw(all, n + 1, s);
        if (!bf16) return launch_gemm_f32_batch(a, n, s);
        return n > 1 ? launch_gemm_bf16_wgrads(a, n, s) : launch_gemm_bf16(a[0], s);
    });
    if (e != hipSuccess) return hip_fail(e, cola_kernel_name(kc));
    if (sp.splits > 1) {
        e = timed(COLA_KC_REDUCE, 0.0, elems * 4.0 * (sp.splits + 1), s,
                  [&] { return launch_reduce(red, n, sp.splits, s); });
        if (e != hipSuccess) return hip_fail(e, "reduce");
    }
    return COLA_OK;
}

template <class F>
int guarded(F&& f) {
    try {
        return f();
    } catch (const std::bad_alloc&) {
        snprintf(g_err, sizeof(g_err), "host allocation failed");
        return COLA_ERR_HIP;
    } catch (...) {
        snprintf(g_err, sizeof(g_err), "unexpected host exception");
        return COLA_ERR_HIP;
    }
}

// The gated product of the decoder block's MLP fused into a GEMM epilogue
// (256 x 256 and smaller tiles, not the streaming family; the caller runs the
// elementwise kernels when *fused comes back false): forward, the last projection
// of a group stores u and m = g u, g being the group's first output; backward, the
// layer's dX = dm GEMM stores dg = dm u and du = dm g instead.  g, u, m, dg and du
// share the row pitch ld.
struct Gate {
    const void* g;
    const void* u;
    int64_t ld;
    void* out;       // m (forward) or dg (backward)
    void* out2;      // du (backward)
    bool* fused;
    bool keep_u;     // forward: the fused epilogue also stores u (else only m)
};

bool gate_fusion_on() { return get_option(OPT_FUSE_GATE) == 1; }

// Forward of one validated layer with its pointers and workspace checked.
// outer >= 0: the both-sigma variant (K2 stores P and Y = sigma_out(P)).
int layer_forward(const Dims& x, FwdPlan p, int act, bool recompute, const void* X, const void* A,
                  const void* B, void* Y, void* Z, void* H, int outer, void* P, char* w, hipStream_t s) {
    void* Hbuf = recompute ? (void*)(w + p.off_h) : H;
    const int64_t ldh = recompute ? p.ldw : x.ldz;
    const double es = (double)x.esize;
    const bool few = x.bf16 && skinny_rows(x.T);
    p.pa = direct(p.pa, few, x.d_in);
    p.pb = direct(p.pb, few, x.r);
    p.px = direct(p.px, few, x.ldx);
    p.ph = direct(p.ph, few, ldh);
    const void *Aw, *Bw, *Xw, *Hw;
    hipError_t e = use_packed(p.pa, A, x.d_in, w, &Aw, s);
    if (e == hipSuccess) e = use_packed(p.pb, B, x.r, w, &Bw, s);
    if (e == hipSuccess) e = use_packed(p.px, X, x.ldx, w, &Xw, s);
    if (e != hipSuccess) return hip_fail(e, "pack_rows");
    const int64_t lda = p.pa.ld, ldb = p.pb.ld;

    // K1: Z = X A^T, H = sigma(Z)
    GemmArgs k1 = make_args(TAG_FWD_Z, x.T, x.r, x.d_in, Xw, p.px.ld, KMAJ, Aw, lda, KMAJ, Z, x.ldz, EPI_Z_H,
                            act);
    k1.aux = Hbuf;
    k1.ldaux = ldh;
    const double b1 = es * ((double)x.T * x.d_in + (double)x.r * x.d_in + 2.0 * x.T * x.r);
    e = timed(COLA_KC_FWD_Z, gemm_flops(x.T, x.r, x.d_in), b1, s, [&] { return gemm(k1, x.bf16, s); });
    if (e != hipSuccess) return hip_fail(e, "fwd_z_sigma");

    // K2: Y = H B^T; with an outer sigma (outer >= 0) K2 stores P = H B^T
    // and Y = sigma_out(P)
    e = use_packed(p.ph, Hbuf, ldh, w, &Hw, s);
    if (e != hipSuccess) return hip_fail(e, "pack_rows");
    GemmArgs k2 = make_args(TAG_FWD_Y, x.T, x.d_out, x.r, Hw, p.ph.ld, KMAJ, Bw, ldb, KMAJ, Y, x.ldy, EPI_STORE,
                            act);
    if (outer >= 0) {
        k2 = make_args(TAG_FWD_YP, x.T, x.d_out, x.r, Hw, p.ph.ld, KMAJ, Bw, ldb, KMAJ, P, x.ldy, EPI_Z_H, outer);
        k2.aux = Y;
        k2.ldaux = x.ldy;
    }
    const double b2 = es * ((double)x.T * x.r + (double)x.d_out * x.r + (double)x.T * x.d_out *
                            (outer >= 0 ? 2.0 : 1.0));
    e = timed(COLA_KC_FWD_Y, gemm_flops(x.T, x.d_out, x.r), b2, s, [&] { return gemm(k2, x.bf16, s); });
    if (e != hipSuccess) return hip_fail(e, "fwd_y");
    return COLA_OK;
}

// Backward of one validated layer with a non-empty batch, its pointers and
// workspace checked against the plan p.
int layer_backward(const Dims& x, const BwdPlan& p, int act, bool recompute, const void* dY_in, const void* X_in,
                   const void* Z, const void* H, const void* A, const void* B, void* dX, float* dA, float* dB,
                   char* w, hipStream_t s, const Gate* gate = nullptr) {
    void* dZ = w + p.off_dz;
    const double es = (double)x.esize;
    const void *Aw, *Bw, *X, *dY, *Hbuf;
    hipError_t e = use_packed(p.wa, A, x.d_in, w, &Aw, s);
    if (e == hipSuccess) e = use_packed(p.wb, B, x.r, w, &Bw, s);
    if (e == hipSuccess) e = use_packed(p.px, X_in, x.ldx, w, &X, s);
    if (e == hipSuccess) e = use_packed(p.py, dY_in, x.ldy, w, &dY, s);
    if (e == hipSuccess) e = use_packed(p.ph, recompute ? (const void*)(w + p.off_h) : H, recompute ? p.ldw : x.ldz, w,
                                        &Hbuf, s);
    if (e != hipSuccess) return hip_fail(e, "pack_rows");
    const int64_t lda = p.wa.ld, ldb = p.wb.ld, ldx = p.px.ld, ldy = p.py.ld, ldh = p.ph.ld;

    // K3: dZ = (dY B) (.) sigma'(Z); CoLA-M regenerates H = sigma(Z) here
    GemmArgs k3 = make_args(TAG_BWD_DZ, x.T, x.r, x.d_out, dY, ldy, KMAJ, Bw, ldb, MNMAJ, dZ, p.ldw, EPI_DZ,
                            act);
    k3.zin = Z;
    k3.ldzin = x.ldz;
    k3.aux = recompute ? (void*)(w + p.off_h) : nullptr;
    k3.ldaux = p.ldw;
    const double b3 = es * ((double)x.T * x.d_out + (double)x.d_out * x.r +
                            (double)x.T * x.r * (recompute ? 3.0 : 2.0));
    e = timed(COLA_KC_BWD_DZ, gemm_flops(x.T, x.r, x.d_out), b3, s, [&] { return gemm(k3, x.bf16, s); });
    if (e != hipSuccess) return hip_fail(e, "bwd_dz");

    // K4: dX = dZ A (or, gated, dg = dm u and du = dm g with dm = dZ A)
    GemmArgs k4 = make_args(TAG_BWD_DX, x.T, x.d_in, x.r, dZ, p.ldw, KMAJ, Aw, lda, MNMAJ, dX, x.ldx, EPI_STORE,
                            act);
    double b4 = es * ((double)x.T * x.r + (double)x.r * x.d_in + (double)x.T * x.d_in);
    if (gate) {
        GemmArgs kg = make_args(TAG_BWD_DXG, x.T, x.d_in, x.r, dZ, p.ldw, KMAJ, Aw, lda, MNMAJ, gate->out, gate->ld,
                                EPI_DGATE, act);
        kg.zin = gate->g;
        kg.ldzin = gate->ld;
        kg.zin2 = gate->u;
        kg.ldzin2 = gate->ld;
        kg.aux = gate->out2;
        kg.ldaux = gate->ld;
        *gate->fused = x.bf16 && gate_fusion_on() && fused_epilogue_takes(kg);
        if (*gate->fused) {
            k4 = kg;
            b4 = es * ((double)x.T * x.r + (double)x.r * x.d_in + 4.0 * x.T * x.d_in);
        }
    }
    const DxProd dxp{k4, b4};
    const bool alone = k4.epi != EPI_STORE;                    // the gated products have a launch of their own
    if (alone) {
        const int st = launch_dx(x.bf16, dxp, s);
        if (st != COLA_OK) return st;
    }
    const DxProd* const with = alone ? nullptr : &dxp;

    // K5: dA = dZ^T X ; K6: dB = dY^T H  (+ K7 fixed-order reductions); one launch
    // for both where planned
    const WProd wp[2] = {{x.r, x.d_in, dZ, X, p.ldw, ldx, dA, reinterpret_cast<float*>(w + p.off_pa), COLA_KC_BWD_DA},
                         {x.d_out, x.r, dY, Hbuf, ldy, ldh, dB, reinterpret_cast<float*>(w + p.off_pb), COLA_KC_BWD_DB}};
    if (p.pair) return wgrads(x.bf16, x.T, p.sa, wp, 2, s, with);
    const int st = wgrads(x.bf16, x.T, p.sa, wp, 1, s, with);
    return st != COLA_OK ? st : wgrads(x.bf16, x.T, p.sb, wp + 1, 1, s);
}

// dA = dB = 0 for an empty batch (the token sums are empty).
int zero_weight_grads(const Dims& x, float* dA, float* dB, hipStream_t s) {
    hipError_t e = timed(COLA_KC_FILL, 0.0, 4.0 * x.r * x.d_in, s,
                         [&] { return launch_fill_zero(dA, x.r * x.d_in, s); });
    if (e == hipSuccess)
        e = timed(COLA_KC_FILL, 0.0, 4.0 * x.d_out * x.r, s, [&] { return launch_fill_zero(dB, x.d_out * x.r, s); });
    return e == hipSuccess ? COLA_OK : hip_fail(e, "fill_zero");
}

int bwd_checked(const cola_desc* desc, const void* dY, const void* X, const void* Z, const void* H, const void* A,
                const void* B, void* dX, float* dA, float* dB, void* ws, size_t ws_bytes, cola_stream_t stream,
                const Gate* gate) {
    Dims x;
    int st = check_desc(desc, &x);
    if (st != COLA_OK) return st;
    const bool recompute = desc->recompute == 1;
    if (recompute ? (H != nullptr) : (H == nullptr && x.T > 0)) return COLA_ERR_INVALID_ARG;
    if (!dA || !dB) return COLA_ERR_INVALID_ARG;
    if (gate) *gate->fused = false;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (x.T == 0) return zero_weight_grads(x, dA, dB, s);
    if (!dY || !X || !Z || !A || !B || !dX) return COLA_ERR_INVALID_ARG;
    const BwdPlan p = fitting(ws_bytes, [&](unsigned copies) { return plan_bwd(x, recompute, copies); });
    if (!ws || ws_bytes < p.total) return COLA_ERR_WORKSPACE;
    return layer_backward(x, p, desc->act, recompute, dY, X, Z, H, A, B, dX, dA, dB,
                          reinterpret_cast<char*>(ws), s, gate);
}

// Workspace of the both-sigma backward: the layer's, then dP = dY sigma_out'(P).
struct OuterPlan {
    int64_t ldg;
    size_t off_g, total;
    BwdPlan bwd;          // of the layer, which reads dP
};

OuterPlan plan_outer_bwd(const Dims& x, bool recompute, unsigned copies = kAllCopies) {
    OuterPlan o;
    o.ldg = line_pitch(x.bf16, x.d_out);
    Dims dp = x;
    dp.ldy = o.ldg;
    o.bwd = plan_bwd(dp, recompute, copies);
    o.off_g = o.bwd.total;
    o.total = x.T == 0 ? 0 : o.off_g + align256((size_t)x.T * (size_t)o.ldg * x.esize);
    return o;
}

}  // namespace

// ---- hooks for the other translation units (the block path) ----
namespace cola {

hipError_t timed_call(int kc, double flops, double bytes, hipStream_t s, hipError_t (*fn)(void*), void* ctx) {
    return timed(kc, flops, bytes, s, [&] { return fn(ctx); });
}

int set_hip_error(hipError_t e, const char* where) { return hip_fail(e, where); }

hipError_t launch_up_projection(int64_t T, int64_t d_out, int64_t r, const void* H, int64_t ldh, const void* B,
                                void* Y, int64_t ldy, hipStream_t s, const void* g, void* m, bool* fused) {
    GemmArgs k2 = make_args(TAG_FWD_Y, T, d_out, r, H, ldh, KMAJ, B, r, KMAJ, Y, ldy, EPI_STORE, 0);
    double bytes = 2.0 * ((double)T * r + (double)d_out * r + (double)T * d_out);
    if (fused) {
        GemmArgs kg = make_args(TAG_FWD_YG, T, d_out, r, H, ldh, KMAJ, B, r, KMAJ, Y, ldy, EPI_GATE, 0);
        kg.zin = g;
        kg.ldzin = ldy;
        kg.aux = m;
        kg.ldaux = ldy;
        *fused = gate_fusion_on() && fused_epilogue_takes(kg);
        if (*fused) {
            k2 = kg;
            bytes = 2.0 * ((double)T * r + (double)d_out * r + 3.0 * T * d_out);
        }
    }
    return timed(COLA_KC_FWD_Y, gemm_flops(T, d_out, r), bytes, s, [&] { return gemm(k2, true, s); });
}

}  // namespace cola

extern "C" {

int cola_abi_version(void) { return COLA_ABI_VERSION; }

int cola_set_option(int option, int value) {
    static_assert((int)COLA_OPT_STREAM_ONLY == (int)OPT_STREAM_ONLY && (int)COLA_OPT_WGRAD_PAIR == (int)OPT_WGRAD_PAIR &&
                      (int)COLA_OPT_FUSE_GATE == (int)OPT_FUSE_GATE && (int)COLA_OPT_TILE == (int)OPT_TILE,
                  "option numbering");
    return set_option(option, value) == 0 ? COLA_OK : COLA_ERR_INVALID_ARG;
}

int cola_get_option(int option) { return get_option(option); }

const char* cola_strerror(int status) {
    switch (status) {
        case COLA_OK: return "success";
        case COLA_ERR_INVALID_ARG: return "invalid argument (NULL pointer, bad enum, or H/recompute mismatch)";
        case COLA_ERR_BAD_SHAPE: return "bad shape (dimension < 1, T < 0, ld < width, or size overflow)";
        case COLA_ERR_WORKSPACE: return "workspace too small";
        case COLA_ERR_HIP: return g_err[0] ? g_err : "HIP error";
        case COLA_ERR_UNSUPPORTED: return "unsupported combination";
        case COLA_ERR_SCRATCH: return "the call needs more than the library's static scratch (COLA_SCRATCH_BYTES)";
        default: return "unknown status";
    }
}

const char* cola_kernel_name(int kc) {
    static const char* names[COLA_KC_COUNT] = {
        "fwd_z_sigma", "fwd_y", "bwd_dz", "bwd_dx", "bwd_da", "bwd_db",
        "reduce_splits", "dense_fwd", "dense_dx", "dense_dw", "fill_zero", "infer_h", "outer_grad",
        "bwd_da_db", "attn_fwd", "attn_bwd", "norm", "norm_bwd", "pointwise"};
    if (kc < 0 || kc >= COLA_KC_COUNT) return "invalid";
    return names[kc];
}

size_t cola_workspace_bytes(const cola_desc* desc, int phase) {
    Dims x;
    if (check_desc(desc, &x) != COLA_OK) return 0;
    const unsigned copies = phase_copies(&phase);
    if (phase == 0) return plan_fwd(x, desc->recompute == 1, copies).total;
    if (phase == 1) return plan_bwd(x, desc->recompute == 1, copies).total;
    if (phase == 2) return plan_fwd(x, true, copies).total;     // inference: H in the workspace, as CoLA-M's forward
    if (phase == 3) return plan_outer_bwd(x, desc->recompute == 1, copies).total;
    return 0;
}

int cola_fwd(const cola_desc* desc, const void* X, const void* A, const void* B, void* Y, void* Z,
             void* H, void* ws, size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        Dims x;
        int st = check_desc(desc, &x);
        if (st != COLA_OK) return st;
        const bool recompute = desc->recompute == 1;
        // CoLA-M never takes H; CoLA needs it unless the batch is empty
        if (recompute ? (H != nullptr) : (H == nullptr && x.T > 0)) return COLA_ERR_INVALID_ARG;
        if (x.T == 0) return COLA_OK;
        if (!X || !A || !B || !Y || !Z) return COLA_ERR_INVALID_ARG;
        const FwdPlan p = fitting(ws ? ws_bytes : 0, [&](unsigned copies) { return plan_fwd(x, recompute, copies); });
        if (p.total > 0 && (!ws || ws_bytes < p.total)) return COLA_ERR_WORKSPACE;
        return layer_forward(x, p, desc->act, recompute, X, A, B, Y, Z, H, -1, nullptr, reinterpret_cast<char*>(ws),
                             reinterpret_cast<hipStream_t>(stream));
    });
}

int cola_fwd_outer(const cola_desc* desc, int outer_act, const void* X, const void* A, const void* B, void* Y,
                   void* P, void* Z, void* H, void* ws, size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        Dims x;
        int st = check_desc(desc, &x);
        if (st != COLA_OK) return st;
        if (!valid_act(outer_act)) return COLA_ERR_INVALID_ARG;
        const bool recompute = desc->recompute == 1;
        if (recompute ? (H != nullptr) : (H == nullptr && x.T > 0)) return COLA_ERR_INVALID_ARG;
        if (x.T == 0) return COLA_OK;
        if (!X || !A || !B || !Y || !P || !Z) return COLA_ERR_INVALID_ARG;
        const FwdPlan p = fitting(ws ? ws_bytes : 0, [&](unsigned copies) { return plan_fwd(x, recompute, copies); });
        if (p.total > 0 && (!ws || ws_bytes < p.total)) return COLA_ERR_WORKSPACE;
        return layer_forward(x, p, desc->act, recompute, X, A, B, Y, Z, H, outer_act, P, reinterpret_cast<char*>(ws),
                             reinterpret_cast<hipStream_t>(stream));
    });
}

int cola_bwd(const cola_desc* desc, const void* dY, const void* X, const void* Z, const void* H,
             const void* A, const void* B, void* dX, float* dA, float* dB, void* ws, size_t ws_bytes,
             cola_stream_t stream) {
    return guarded([&]() -> int { return bwd_checked(desc, dY, X, Z, H, A, B, dX, dA, dB, ws, ws_bytes, stream, nullptr); });
}

// ---------------------------------------------------------------------------
// backward without a caller workspace: the library's static device scratch
// ---------------------------------------------------------------------------
}  // extern "C"

namespace {

// The workspace of cola_bwd_scratch: one array per GPU, placed by the code
// object loader and held until the process ends.  In host code `scratch` is
// a host-side stand-in, not a device address: kernels get the address that
// hipGetSymbolAddress returns for the current device, kept per device.
static __device__ __align__(256) unsigned char scratch[COLA_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;

struct ScratchPtrs {
    std::mutex mu;
    void* ptr[kMaxDevices] = {};
};

ScratchPtrs& scratch_ptrs() {
    static ScratchPtrs* s = new ScratchPtrs();   // never destroyed
    return *s;
}

// The size by which cola_bwd_scratch accepts a call: dZ, H (CoLA-M), repacked
// weights and the room for partials, which the lean plan never exceeds.
size_t scratch_demand(const Dims& x, bool recompute) {
    if (x.T == 0) return 0;
    const WShape w[2] = {{x.r, x.d_in}, {x.d_out, x.r}};
    size_t total = align256((size_t)x.T * (size_t)line_pitch(x.bf16, x.r) * x.esize) * (recompute ? 2 : 1);
    for (int i = 0; i < 2; ++i) total += plan_weight(x.bf16, w[i].M, w[i].N, 0).bytes;
    if (get_option(OPT_WGRAD_PAIR) == 1) return total + partial_room(x.bf16, w, 2, x.T);
    return total + partial_room(x.bf16, w, 1, x.T) + partial_room(x.bf16, w + 1, 1, x.T);
}

// Device address of this device's scratch (looked up once per device, with
// that device current).
int scratch_of_current_device(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) {
        snprintf(g_err, sizeof(g_err), "device %d beyond the %d the scratch table holds", dev, kMaxDevices);
        return COLA_ERR_HIP;
    }
    ScratchPtrs& t = scratch_ptrs();
    std::lock_guard<std::mutex> lock(t.mu);
    if (!t.ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p) {
            snprintf(g_err, sizeof(g_err), "hipGetSymbolAddress(scratch) returned NULL");
            return COLA_ERR_HIP;
        }
        t.ptr[dev] = p;
    }
    *out = t.ptr[dev];
    return COLA_OK;
}

}  // namespace

extern "C" {

int cola_bwd_scratch(const cola_desc* desc, const void* dY, const void* X, const void* Z, const void* H,
                     const void* A, const void* B, void* dX, float* dA, float* dB, cola_stream_t stream) {
    return guarded([&]() -> int {
        Dims x;
        int st = check_desc(desc, &x);
        if (st != COLA_OK) return st;
        const bool recompute = desc->recompute == 1;
        if (recompute ? (H != nullptr) : (H == nullptr && x.T > 0)) return COLA_ERR_INVALID_ARG;
        if (!dA || !dB) return COLA_ERR_INVALID_ARG;
        hipStream_t s = reinterpret_cast<hipStream_t>(stream);
        if (x.T == 0) return zero_weight_grads(x, dA, dB, s);
        if (!dY || !X || !Z || !A || !B || !dX) return COLA_ERR_INVALID_ARG;
        if (scratch_demand(x, recompute) > COLA_SCRATCH_BYTES) return COLA_ERR_SCRATCH;
        const BwdPlan p = fitting(COLA_SCRATCH_BYTES, [&](unsigned copies) { return plan_bwd(x, recompute, copies); });
        if (p.total > COLA_SCRATCH_BYTES) return COLA_ERR_SCRATCH;
        void* w = nullptr;
        st = scratch_of_current_device(&w);
        if (st != COLA_OK) return st;
        return layer_backward(x, p, desc->act, recompute, dY, X, Z, H, A, B, dX, dA, dB,
                              reinterpret_cast<char*>(w), s);
    });
}

int cola_bwd_outer(const cola_desc* desc, int outer_act, const void* dY, const void* P, const void* X,
                   const void* Z, const void* H, const void* A, const void* B, void* dX, float* dA, float* dB,
                   void* ws, size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        Dims x;
        int st = check_desc(desc, &x);
        if (st != COLA_OK) return st;
        if (!valid_act(outer_act)) return COLA_ERR_INVALID_ARG;
        const bool recompute = desc->recompute == 1;
        if (recompute ? (H != nullptr) : (H == nullptr && x.T > 0)) return COLA_ERR_INVALID_ARG;
        if (!dA || !dB) return COLA_ERR_INVALID_ARG;
        hipStream_t s = reinterpret_cast<hipStream_t>(stream);
        if (x.T == 0) return zero_weight_grads(x, dA, dB, s);
        if (!dY || !P || !X || !Z || !A || !B || !dX) return COLA_ERR_INVALID_ARG;
        const OuterPlan o = fitting(ws_bytes, [&](unsigned copies) { return plan_outer_bwd(x, recompute, copies); });
        if (!ws || ws_bytes < o.total) return COLA_ERR_WORKSPACE;
        char* w = reinterpret_cast<char*>(ws);
        // dP = dY (.) sigma_out'(P), rounded to the storage dtype like dZ
        void* dP = w + o.off_g;
        const double bytes = (double)x.esize * 3.0 * (double)x.T * (double)x.d_out;
        hipError_t e = timed(COLA_KC_OUTER_GRAD, 0.0, bytes, s, [&] {
            return launch_outer_grad(x.bf16, dY, x.ldy, P, x.ldy, dP, o.ldg, x.T, x.d_out, outer_act, s);
        });
        if (e != hipSuccess) return hip_fail(e, "outer_grad");
        return layer_backward(x, o.bwd, desc->act, recompute, dP, X, Z, H, A, B, dX, dA, dB, w, s);
    });
}

// ---------------------------------------------------------------------------
// dense baseline
// ---------------------------------------------------------------------------
static int check_dense(const dense_desc* d, Dims* out) {
    if (!d) return COLA_ERR_INVALID_ARG;
    cola_desc c{};
    c.T = d->T; c.d_in = d->d_in; c.d_out = d->d_out; c.r = 1;
    c.ldx = d->ldx; c.ldy = d->ldy; c.ldz = 0;
    c.dtype = d->dtype; c.act = COLA_ACT_IDENTITY; c.recompute = 0;
    return check_desc(&c, out);
}

// Workspace of the dense path: [split-K partials of dW (phase 1)] [W repack].
struct DensePlan {
    Split sp;
    size_t parts;
    Pack pw;
    size_t total;
};

static DensePlan plan_dense(const Dims& x, int phase) {
    DensePlan p;
    const WShape w{x.d_out, x.d_in};
    p.sp = plan_split(x.bf16, &w, 1, x.T, !pitch16(x.ldx) || !pitch16(x.ldy));
    p.parts = (phase == 1 && p.sp.splits > 1) ? align256((size_t)p.sp.splits * (size_t)(x.d_out * x.d_in) * 4) : 0;
    p.pw = plan_weight(x.bf16, x.d_out, x.d_in, p.parts);
    p.total = p.pw.off + p.pw.bytes;
    if (x.T == 0) p.total = 0;
    return p;
}

size_t dense_workspace_bytes(const dense_desc* desc, int phase) {
    Dims x;
    if (check_dense(desc, &x) != COLA_OK) return 0;
    if (phase != 0 && phase != 1) return 0;
    return plan_dense(x, phase).total;
}

int dense_fwd(const dense_desc* desc, const void* X, const void* W, void* Y, void* ws, size_t ws_bytes,
              cola_stream_t stream) {
    return guarded([&]() -> int {
        Dims x;
        int st = check_dense(desc, &x);
        if (st != COLA_OK) return st;
        if (x.T == 0) return COLA_OK;
        if (!X || !W || !Y) return COLA_ERR_INVALID_ARG;
        const DensePlan p = plan_dense(x, 0);
        if (p.total > 0 && (!ws || ws_bytes < p.total)) return COLA_ERR_WORKSPACE;
        hipStream_t s = reinterpret_cast<hipStream_t>(stream);
        const void* Ww;
        hipError_t e = use_packed(p.pw, W, x.d_in, reinterpret_cast<char*>(ws), &Ww, s);
        const int64_t ldw = p.pw.ld;
        if (e != hipSuccess) return hip_fail(e, "pack_rows");
        GemmArgs a = make_args(TAG_DENSE_FWD, x.T, x.d_out, x.d_in, X, x.ldx, KMAJ, Ww, ldw, KMAJ, Y, x.ldy, EPI_STORE, 0);
        const double b = (double)x.esize * ((double)x.T * x.d_in + (double)x.d_out * x.d_in + (double)x.T * x.d_out);
        e = timed(COLA_KC_DENSE_FWD, gemm_flops(x.T, x.d_out, x.d_in), b, s, [&] { return gemm(a, x.bf16, s); });
        return e == hipSuccess ? COLA_OK : hip_fail(e, "dense_fwd");
    });
}

int dense_bwd(const dense_desc* desc, const void* dY, const void* X, const void* W, void* dX, float* dW,
              void* ws, size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        Dims x;
        int st = check_dense(desc, &x);
        if (st != COLA_OK) return st;
        if (!dW) return COLA_ERR_INVALID_ARG;
        hipStream_t s = reinterpret_cast<hipStream_t>(stream);
        if (x.T == 0) {
            hipError_t e = timed(COLA_KC_FILL, 0.0, 4.0 * x.d_out * x.d_in, s,
                                 [&] { return launch_fill_zero(dW, x.d_out * x.d_in, s); });
            return e == hipSuccess ? COLA_OK : hip_fail(e, "fill_zero");
        }
        if (!dY || !X || !W || !dX) return COLA_ERR_INVALID_ARG;
        const DensePlan p = plan_dense(x, 1);
        if (p.total > 0 && (!ws || ws_bytes < p.total)) return COLA_ERR_WORKSPACE;
        char* w = reinterpret_cast<char*>(ws);
        const void* Ww;
        hipError_t e = use_packed(p.pw, W, x.d_in, w, &Ww, s);
        const int64_t ldw = p.pw.ld;
        if (e != hipSuccess) return hip_fail(e, "pack_rows");
        GemmArgs a = make_args(TAG_DENSE_DX, x.T, x.d_in, x.d_out, dY, x.ldy, KMAJ, Ww, ldw, MNMAJ, dX, x.ldx, EPI_STORE, 0);
        const double b = (double)x.esize * ((double)x.T * x.d_out + (double)x.d_out * x.d_in + (double)x.T * x.d_in);
        e = timed(COLA_KC_DENSE_DX, gemm_flops(x.T, x.d_in, x.d_out), b, s, [&] { return gemm(a, x.bf16, s); });
        if (e != hipSuccess) return hip_fail(e, "dense_dx");
        const WProd wp{x.d_out, x.d_in, dY, X, x.ldy, x.ldx, dW, reinterpret_cast<float*>(w), COLA_KC_DENSE_DW};
        return wgrads(x.bf16, x.T, p.sp, &wp, 1, s);
    });
}

// ---------------------------------------------------------------------------
// timing API
// ---------------------------------------------------------------------------
int cola_timing_enable(int on) {
    return guarded([&]() -> int {
        TimingState& t = timing();
        std::lock_guard<std::mutex> lock(t.mu);
        t.on = on != 0;
        return COLA_OK;
    });
}

int cola_timing_reset(void) {
    return guarded([&]() -> int {
        TimingState& t = timing();
        std::lock_guard<std::mutex> lock(t.mu);
        hipError_t e = drain(t);
        for (int k = 0; k < COLA_KC_COUNT; ++k) {
            t.launches[k] = 0; t.ms[k] = 0; t.flops[k] = 0; t.bytes[k] = 0;
        }
        return e == hipSuccess ? COLA_OK : hip_fail(e, "timing_reset");
    });
}

int cola_timing_read(int kc, int64_t* launches, double* ms, double* flops, double* bytes) {
    if (kc < 0 || kc >= COLA_KC_COUNT || !launches || !ms || !flops || !bytes) return COLA_ERR_INVALID_ARG;
    return guarded([&]() -> int {
        TimingState& t = timing();
        std::lock_guard<std::mutex> lock(t.mu);
        hipError_t e = drain(t);
        if (e != hipSuccess) return hip_fail(e, "timing_read");
        *launches = t.launches[kc];
        *ms = t.ms[kc];
        *flops = t.flops[kc];
        *bytes = t.bytes[kc];
        return COLA_OK;
    });
}

}  // extern "C"

// ---------------------------------------------------------------------------
// grouped projections that read the same input
// ---------------------------------------------------------------------------
namespace {

struct GDims {
    int64_t T, d_in, ldx, ldz, R;
    int n;
    int64_t r[COLA_GROUP_MAX], d_out[COLA_GROUP_MAX], ldy[COLA_GROUP_MAX], off[COLA_GROUP_MAX];
    bool bf16;
    size_t esize;
};

int check_group(const cola_group_desc* d, GDims* out) {
    if (!d) return COLA_ERR_INVALID_ARG;
    if (d->n < 1 || d->n > COLA_GROUP_MAX) return COLA_ERR_INVALID_ARG;
    GDims g{};
    g.n = d->n;
    g.R = 0;
    for (int p = 0; p < g.n; ++p) {
        // each projection must be a valid single layer (enums, shapes, pitches)
        cola_desc c{};
        c.T = d->T; c.d_in = d->d_in; c.d_out = d->d_out[p]; c.r = d->r[p];
        c.ldx = d->ldx; c.ldy = d->ldy[p]; c.ldz = 0;
        c.dtype = d->dtype; c.act = d->act; c.recompute = d->recompute;
        Dims x;
        const int st = check_desc(&c, &x);
        if (st != COLA_OK) return st;
        g.r[p] = x.r; g.d_out[p] = x.d_out; g.ldy[p] = x.ldy; g.off[p] = g.R;
        g.R += x.r;
        g.T = x.T; g.d_in = x.d_in; g.ldx = x.ldx; g.bf16 = x.bf16; g.esize = x.esize;
    }
    if (g.R > kMaxDim) return COLA_ERR_BAD_SHAPE;
    g.ldz = d->ldz ? d->ldz : g.R;
    if (g.ldz < g.R || g.ldz > kMaxPitch) return COLA_ERR_BAD_SHAPE;
    if ((double)g.T * (double)g.ldz > 4.0e18 || (double)g.R * (double)g.d_in > 4.0e18) return COLA_ERR_BAD_SHAPE;
    *out = g;
    return COLA_OK;
}

// Workspace: [H_all copy (CoLA-M)] [repacked A_all] [repacked B_p ...] [repacked X]
// [repacked H_p ...] (token rows where they are not 16-byte aligned)
struct GFwdPlan {
    int64_t ldw;
    size_t off_h, total;
    Pack pa, pb[COLA_GROUP_MAX], px, ph[COLA_GROUP_MAX];
};

// H_p starts on a 16-byte boundary in every row (columns off[p] .. of H_all).
bool group_h_aligned(const GDims& g, bool recompute, int p) {
    return g.off[p] % 8 == 0 && (recompute || pitch16(g.ldz));
}

GFwdPlan plan_group_fwd(const GDims& g, bool recompute, unsigned copies = kAllCopies) {
    GFwdPlan p;
    p.ldw = line_pitch(g.bf16, g.R);
    p.off_h = 0;
    const size_t hbytes = recompute ? align256((size_t)g.T * (size_t)p.ldw * g.esize) : 0;
    p.pa = plan_weight(g.bf16, g.R, g.d_in, hbytes);
    size_t next = p.pa.off + p.pa.bytes;
    for (int q = 0; q < g.n; ++q) {
        p.pb[q] = plan_weight(g.bf16, g.d_out[q], g.r[q], next);
        next = p.pb[q].off + p.pb[q].bytes;
    }
    if (!g.bf16) copies = 0;
    p.px = plan_pack((copies & COPY_X) && !pitch16(g.ldx), g.T, g.d_in, g.ldx, next);
    next = p.px.off + p.px.bytes;
    for (int q = 0; q < g.n; ++q) {
        p.ph[q] = plan_pack((copies & COPY_H) && !group_h_aligned(g, recompute, q), g.T, g.r[q],
                            recompute ? p.ldw : g.ldz, next);
        next = p.ph[q].off + p.ph[q].bytes;
    }
    p.total = g.T == 0 ? 0 : next;
    return p;
}

// The weight gradients of a group are the products w = 0 (dA_all, R x d_in)
// and w = 1 + p (dB_p, d_out_p x r_p), all over K = T.  They run in sets of up to
// kWSet, w = 0 .. 3, 4 .. 7, 8: one launch with one split for a set, or one launch
// each where sets are off.  Their tiles together fill the CUs with
// fewer splits (gate and up of the 350M shape at 32768 tokens: dA with one dB and
// the other dB apart 197 us with their reductions, the three together 141).
// Workspace: [dZ_all] [H_all (CoLA-M)] [partials of the set's products, reused set
// after set] [repacked A_all] [repacked B_p ...] [repacked X] [repacked dY_p, H_p ...].
struct GBwdPlan {
    int64_t ldw;
    size_t off_dz, off_h, off_p[kWSet], total;
    int nw;                                // 1 + number of projections
    Split sp[COLA_GROUP_MAX + 1];          // split of each product (shared within a launched set)
    bool set[COLA_GROUP_MAX + 1];          // the set starting at w runs in one launch
    Pack wa, wb[COLA_GROUP_MAX], px, py[COLA_GROUP_MAX], ph[COLA_GROUP_MAX];
};

// Shape of weight-gradient product w of a group.
WShape group_wgrad_shape(const GDims& g, int w) {
    return w == 0 ? WShape{g.R, g.d_in} : WShape{g.d_out[w - 1], g.r[w - 1]};
}

GBwdPlan plan_group_bwd(const GDims& g, bool recompute, unsigned copies = kAllCopies) {
    GBwdPlan p;
    p.ldw = line_pitch(g.bf16, g.R);
    const size_t zbytes = align256((size_t)g.T * (size_t)p.ldw * g.esize);
    p.off_dz = 0;
    p.off_h = zbytes;
    size_t next = p.off_h + (recompute ? zbytes : 0);
    if (!g.bf16) copies = 0;
    p.nw = g.n + 1;
    size_t pb[kWSet] = {};
    for (int w0 = 0; w0 < p.nw; w0 += kWSet) {
        const int cnt = p.nw - w0 < kWSet ? p.nw - w0 : kWSet;
        WShape w[kWSet];
        for (int k = 0; k < cnt; ++k) w[k] = group_wgrad_shape(g, w0 + k);
        p.set[w0] = cnt > 1 && pair_wgrads(g.bf16);
        if (p.set[w0]) p.sp[w0] = plan_split(g.bf16, w, cnt, g.T);
        for (int k = 0; k < cnt; ++k) {
            Split& sp = p.sp[w0 + k];
            sp = p.set[w0] ? p.sp[w0] : plan_split(g.bf16, w + k, 1, g.T);
            const size_t b = partial_bytes(w + k, 1, sp.splits);
            if (b > pb[k]) pb[k] = b;
        }
    }
    for (int k = 0; k < kWSet; ++k) {
        p.off_p[k] = next;
        next += pb[k];
    }
    p.wa = plan_weight(g.bf16, g.R, g.d_in, next);
    next = p.wa.off + p.wa.bytes;
    for (int q = 0; q < g.n; ++q) {
        p.wb[q] = plan_weight(g.bf16, g.d_out[q], g.r[q], next);
        next = p.wb[q].off + p.wb[q].bytes;
    }
    p.px = plan_pack((copies & COPY_X) && !pitch16(g.ldx), g.T, g.d_in, g.ldx, next);
    next = p.px.off + p.px.bytes;
    for (int q = 0; q < g.n; ++q) {
        p.py[q] = plan_pack((copies & COPY_DY) && !pitch16(g.ldy[q]), g.T, g.d_out[q], g.ldy[q], next);
        p.ph[q] = plan_pack((copies & COPY_H) && !group_h_aligned(g, recompute, q), g.T, g.r[q],
                            recompute ? p.ldw : g.ldz, p.py[q].off + p.py[q].bytes);
        next = p.ph[q].off + p.ph[q].bytes;
    }
    p.total = g.T == 0 ? 0 : next;
    return p;
}

}  // namespace

extern "C" {

size_t cola_group_workspace_bytes(const cola_group_desc* desc, int phase) {
    GDims g;
    if (check_group(desc, &g) != COLA_OK) return 0;
    const unsigned copies = phase_copies(&phase);
    if (phase == 0) return plan_group_fwd(g, desc->recompute == 1, copies).total;
    if (phase == 1) return plan_group_bwd(g, desc->recompute == 1, copies).total;
    if (phase == 2) return plan_group_fwd(g, true, copies).total;
    return 0;
}

}  // extern "C"

namespace {

// Forward of a validated group with the pointers checked.  Z_all == NULL is
// the inference forward: K1 stores only H (into the workspace), nothing is
// kept for a backward pass.
int group_forward(const GDims& g, GFwdPlan p, int act, const void* X_in, const void* A_all,
                  const void* const* B, void* const* Y, void* Z_all, void* H_all, bool h_in_ws, char* w, hipStream_t s,
                  const Gate* gate = nullptr) {
    char* Hbuf = h_in_ws ? w + p.off_h : reinterpret_cast<char*>(H_all);
    const int64_t ldh = h_in_ws ? p.ldw : g.ldz;
    const double es = (double)g.esize;

    const bool few = g.bf16 && skinny_rows(g.T);
    p.pa = direct(p.pa, few, g.d_in);
    p.px = direct(p.px, few, g.ldx);
    for (int q = 0; q < g.n; ++q) {
        p.pb[q] = direct(p.pb[q], few, g.r[q]);
        p.ph[q] = direct(p.ph[q], few, ldh);
    }
    const void *Aw, *X;
    hipError_t e = use_packed(p.pa, A_all, g.d_in, w, &Aw, s);
    if (e == hipSuccess) e = use_packed(p.px, X_in, g.ldx, w, &X, s);
    if (e != hipSuccess) return hip_fail(e, "pack_rows");
    const int64_t lda = p.pa.ld, ldx = p.px.ld;

    // K1 for every projection at once: Z_all = X A_all^T, H_all = sigma(Z_all)
    if (Z_all) {
        GemmArgs k1 = make_args(TAG_FWD_Z, g.T, g.R, g.d_in, X, ldx, KMAJ, Aw, lda, KMAJ, Z_all, g.ldz, EPI_Z_H,
                                act);
        k1.aux = Hbuf;
        k1.ldaux = ldh;
        const double b1 = es * ((double)g.T * g.d_in + (double)g.R * g.d_in + 2.0 * g.T * g.R);
        e = timed(COLA_KC_FWD_Z, gemm_flops(g.T, g.R, g.d_in), b1, s, [&] { return gemm(k1, g.bf16, s); });
        if (e != hipSuccess) return hip_fail(e, "fwd_z_sigma");
    } else {
        GemmArgs k1 = make_args(TAG_INFER_H, g.T, g.R, g.d_in, X, ldx, KMAJ, Aw, lda, KMAJ, Hbuf, ldh, EPI_H, act);
        const double b1 = es * ((double)g.T * g.d_in + (double)g.R * g.d_in + (double)g.T * g.R);
        e = timed(COLA_KC_INFER_H, gemm_flops(g.T, g.R, g.d_in), b1, s, [&] { return gemm(k1, g.bf16, s); });
        if (e != hipSuccess) return hip_fail(e, "infer_h");
    }

    // K2: Y_p = H_p B_p^T, the projections together
    GemmArgs k2[COLA_GROUP_MAX];
    double f2 = 0.0, b2 = 0.0;
    int n2 = 0;
    for (int q = 0; q < g.n; ++q) {
        const void *Bw, *Hq;
        e = use_packed(p.pb[q], B[q], g.r[q], w, &Bw, s);
        if (e == hipSuccess) e = use_packed(p.ph[q], Hbuf + g.off[q] * g.esize, ldh, w, &Hq, s);
        if (e != hipSuccess) return hip_fail(e, "pack_rows");
        const int64_t ldb = p.pb[q].ld;
        const double fq = gemm_flops(g.T, g.d_out[q], g.r[q]);
        const double bq = es * ((double)g.T * g.r[q] + (double)g.d_out[q] * g.r[q]);
        if (gate && q == g.n - 1) {
            // the last projection also stores m = g u (g: the group's first output)
            GemmArgs kg = make_args(TAG_FWD_YG, g.T, g.d_out[q], g.r[q], Hq, p.ph[q].ld, KMAJ, Bw, ldb, KMAJ, Y[q],
                                    gate->ld, EPI_GATE, act);
            kg.zin = gate->g;
            kg.ldzin = gate->ld;
            kg.aux = gate->out;
            kg.ldaux = gate->ld;
            *gate->fused = g.bf16 && gate_fusion_on() && g.ldy[q] == gate->ld && fused_epilogue_takes(kg);
            if (*gate->fused) {
                if (!gate->keep_u) kg.c = nullptr;
                e = gemms(k2, n2, COLA_KC_FWD_Y, f2, b2, g.bf16, s);      // first: g is one of their outputs
                n2 = 0;
                if (e == hipSuccess)
                    e = timed(COLA_KC_FWD_Y, fq, bq + es * (gate->keep_u ? 3.0 : 2.0) * g.T * g.d_out[q], s,
                              [&] { return gemm(kg, g.bf16, s); });
                if (e != hipSuccess) return hip_fail(e, "fwd_y");
                continue;
            }
        }
        k2[n2++] = make_args(TAG_FWD_Y, g.T, g.d_out[q], g.r[q], Hq, p.ph[q].ld, KMAJ, Bw, ldb, KMAJ, Y[q], g.ldy[q],
                             EPI_STORE, act);
        f2 += fq;
        b2 += bq + es * (double)g.T * g.d_out[q];
    }
    e = gemms(k2, n2, COLA_KC_FWD_Y, f2, b2, g.bf16, s);
    if (e != hipSuccess) return hip_fail(e, "fwd_y");
    return COLA_OK;
}

// The group of one projection that a single-layer descriptor describes.
GDims single_group(const Dims& x) {
    GDims g{};
    g.T = x.T; g.d_in = x.d_in; g.ldx = x.ldx; g.ldz = x.ldz; g.R = x.r; g.n = 1;
    g.r[0] = x.r; g.d_out[0] = x.d_out; g.ldy[0] = x.ldy; g.off[0] = 0;
    g.bf16 = x.bf16; g.esize = x.esize;
    return g;
}

int group_fwd_checked(const cola_group_desc* desc, const void* X, const void* A_all, const void* const* B,
                      void* const* Y, void* Z_all, void* H_all, void* ws, size_t ws_bytes, cola_stream_t stream,
                      const Gate* gate) {
    GDims g;
    int st = check_group(desc, &g);
    if (st != COLA_OK) return st;
    const bool recompute = desc->recompute == 1;
    if (recompute ? (H_all != nullptr) : (H_all == nullptr && g.T > 0)) return COLA_ERR_INVALID_ARG;
    if (gate) *gate->fused = false;
    if (g.T == 0) return COLA_OK;
    if (!X || !A_all || !B || !Y || !Z_all) return COLA_ERR_INVALID_ARG;
    for (int q = 0; q < g.n; ++q)
        if (!B[q] || !Y[q]) return COLA_ERR_INVALID_ARG;
    const GFwdPlan p = fitting(ws ? ws_bytes : 0, [&](unsigned copies) { return plan_group_fwd(g, recompute, copies); });
    if (p.total > 0 && (!ws || ws_bytes < p.total)) return COLA_ERR_WORKSPACE;
    return group_forward(g, p, desc->act, X, A_all, B, Y, Z_all, H_all, recompute, reinterpret_cast<char*>(ws),
                         reinterpret_cast<hipStream_t>(stream), gate);
}

int infer_checked(const GDims& g, int act, const void* X, const void* A_all, const void* const* B, void* const* Y,
                  void* ws, size_t ws_bytes, cola_stream_t stream) {
    if (g.T == 0) return COLA_OK;
    if (!X || !A_all || !B || !Y) return COLA_ERR_INVALID_ARG;
    for (int q = 0; q < g.n; ++q)
        if (!B[q] || !Y[q]) return COLA_ERR_INVALID_ARG;
    const GFwdPlan p = fitting(ws ? ws_bytes : 0, [&](unsigned copies) { return plan_group_fwd(g, true, copies); });
    if (p.total > 0 && (!ws || ws_bytes < p.total)) return COLA_ERR_WORKSPACE;
    return group_forward(g, p, act, X, A_all, B, Y, nullptr, nullptr, true, reinterpret_cast<char*>(ws),
                         reinterpret_cast<hipStream_t>(stream));
}

}  // namespace

extern "C" {

int cola_group_fwd(const cola_group_desc* desc, const void* X, const void* A_all, const void* const* B,
                   void* const* Y, void* Z_all, void* H_all, void* ws, size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        return group_fwd_checked(desc, X, A_all, B, Y, Z_all, H_all, ws, ws_bytes, stream, nullptr);
    });
}

int cola_group_infer(const cola_group_desc* desc, const void* X, const void* A_all, const void* const* B,
                     void* const* Y, void* ws, size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        GDims g;
        const int st = check_group(desc, &g);
        if (st != COLA_OK) return st;
        return infer_checked(g, desc->act, X, A_all, B, Y, ws, ws_bytes, stream);
    });
}

int cola_infer(const cola_desc* desc, const void* X, const void* A, const void* B, void* Y, void* ws,
               size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        Dims x;
        const int st = check_desc(desc, &x);
        if (st != COLA_OK) return st;
        const void* Bs[1] = {B};
        void* Ys[1] = {Y};
        return infer_checked(single_group(x), desc->act, X, A, Bs, Ys, ws, ws_bytes, stream);
    });
}

int cola_group_bwd(const cola_group_desc* desc, const void* const* dY, const void* X_in, const void* Z_all,
                   const void* H_all, const void* A_all, const void* const* B, void* dX, float* dA_all,
                   float* const* dB, void* ws, size_t ws_bytes, cola_stream_t stream) {
    return guarded([&]() -> int {
        GDims g;
        int st = check_group(desc, &g);
        if (st != COLA_OK) return st;
        const bool recompute = desc->recompute == 1;
        if (recompute ? (H_all != nullptr) : (H_all == nullptr && g.T > 0)) return COLA_ERR_INVALID_ARG;
        if (!dA_all || !dB) return COLA_ERR_INVALID_ARG;
        for (int q = 0; q < g.n; ++q)
            if (!dB[q]) return COLA_ERR_INVALID_ARG;
        hipStream_t s = reinterpret_cast<hipStream_t>(stream);
        if (g.T == 0) {
            // empty batch: the token sums are empty
            hipError_t e = timed(COLA_KC_FILL, 0.0, 4.0 * g.R * g.d_in, s,
                                 [&] { return launch_fill_zero(dA_all, g.R * g.d_in, s); });
            for (int q = 0; q < g.n && e == hipSuccess; ++q)
                e = timed(COLA_KC_FILL, 0.0, 4.0 * g.d_out[q] * g.r[q], s,
                          [&] { return launch_fill_zero(dB[q], g.d_out[q] * g.r[q], s); });
            return e == hipSuccess ? COLA_OK : hip_fail(e, "fill_zero");
        }
        if (!dY || !X_in || !Z_all || !A_all || !B || !dX) return COLA_ERR_INVALID_ARG;
        for (int q = 0; q < g.n; ++q)
            if (!dY[q] || !B[q]) return COLA_ERR_INVALID_ARG;
        const GBwdPlan p = fitting(ws_bytes, [&](unsigned copies) { return plan_group_bwd(g, recompute, copies); });
        if (!ws || ws_bytes < p.total) return COLA_ERR_WORKSPACE;

        char* w = reinterpret_cast<char*>(ws);
        char* dZ = w + p.off_dz;
        const char* Hbuf = recompute ? w + p.off_h : reinterpret_cast<const char*>(H_all);
        const int64_t ldh = recompute ? p.ldw : g.ldz;
        const double es = (double)g.esize;
        const void *Aw, *X, *dYw[COLA_GROUP_MAX];
        hipError_t e = use_packed(p.wa, A_all, g.d_in, w, &Aw, s);
        if (e == hipSuccess) e = use_packed(p.px, X_in, g.ldx, w, &X, s);
        for (int q = 0; q < g.n && e == hipSuccess; ++q) e = use_packed(p.py[q], dY[q], g.ldy[q], w, &dYw[q], s);
        if (e != hipSuccess) return hip_fail(e, "pack_rows");
        const int64_t lda = p.wa.ld;

        // K3: dZ_p = (dY_p B_p) (.) sigma'(Z_p)  [+ H_p for CoLA-M], the projections together
        GemmArgs k3[COLA_GROUP_MAX];
        double f3 = 0.0, b3 = 0.0;
        for (int q = 0; q < g.n; ++q) {
            const void* Bw;
            e = use_packed(p.wb[q], B[q], g.r[q], w, &Bw, s);
            if (e != hipSuccess) return hip_fail(e, "pack_rows");
            k3[q] = make_args(TAG_BWD_DZ, g.T, g.r[q], g.d_out[q], dYw[q], p.py[q].ld, KMAJ, Bw, p.wb[q].ld, MNMAJ,
                              dZ + g.off[q] * g.esize, p.ldw, EPI_DZ, desc->act);
            k3[q].zin = reinterpret_cast<const char*>(Z_all) + g.off[q] * g.esize;
            k3[q].ldzin = g.ldz;
            k3[q].aux = recompute ? (void*)(w + p.off_h + g.off[q] * g.esize) : nullptr;
            k3[q].ldaux = p.ldw;
            f3 += gemm_flops(g.T, g.r[q], g.d_out[q]);
            b3 += es * ((double)g.T * g.d_out[q] + (double)g.d_out[q] * g.r[q] +
                        (double)g.T * g.r[q] * (recompute ? 3.0 : 2.0));
        }
        e = gemms(k3, g.n, COLA_KC_BWD_DZ, f3, b3, g.bf16, s);
        if (e != hipSuccess) return hip_fail(e, "bwd_dz");

        // K4 for every projection at once: dX = dZ_all A_all = sum_p dZ_p A_p
        GemmArgs k4 = make_args(TAG_BWD_DX, g.T, g.d_in, g.R, dZ, p.ldw, KMAJ, Aw, lda, MNMAJ, dX, g.ldx, EPI_STORE,
                                desc->act);
        const double b4 = es * ((double)g.T * g.R + (double)g.R * g.d_in + (double)g.T * g.d_in);
        const DxProd dxp{k4, b4};

        // K5 for every projection at once, dA_all = dZ_all^T X (product 0),
        // and K6 per projection, dB_p = dY_p^T H_p (product 1 + p), in sets
        for (int w0 = 0; w0 < p.nw; w0 += kWSet) {
            const int cnt = p.nw - w0 < kWSet ? p.nw - w0 : kWSet;
            WProd wp[kWSet];
            for (int k = 0; k < cnt; ++k) {
                float* part = reinterpret_cast<float*>(w + p.off_p[k]);
                const int q = w0 + k - 1;
                if (q < 0) {
                    wp[k] = WProd{g.R, g.d_in, dZ, X, p.ldw, p.px.ld, dA_all, part, COLA_KC_BWD_DA};
                    continue;
                }
                const void* Hw;                            // CoLA-M: K3 wrote H
                e = use_packed(p.ph[q], Hbuf + g.off[q] * g.esize, ldh, w, &Hw, s);
                if (e != hipSuccess) return hip_fail(e, "pack_rows");
                wp[k] = WProd{g.d_out[q], g.r[q], dYw[q], Hw, p.py[q].ld, p.ph[q].ld, dB[q], part, COLA_KC_BWD_DB};
            }
            if (p.set[w0]) {
                st = wgrads(g.bf16, g.T, p.sp[w0], wp, cnt, s, w0 == 0 ? &dxp : nullptr);
                if (st != COLA_OK) return st;
                continue;
            }
            for (int k = 0; k < cnt; ++k) {
                st = wgrads(g.bf16, g.T, p.sp[w0 + k], wp + k, 1, s, w0 + k == 0 ? &dxp : nullptr);
                if (st != COLA_OK) return st;
            }
        }
        return COLA_OK;
    });
}

}  // extern "C"

// ---- the block's gated-product hooks (block.hpp) ----
namespace cola {

int group_fwd_gated(const cola_group_desc* desc, const void* X, const void* A_all, const void* const* B,
                    void* const* Y, void* Z_all, void* H_all, void* ws, size_t ws_bytes, cola_stream_t stream,
                    const void* g, int64_t ld, void* m, bool* fused, bool keep_u) {
    if (!fused) return COLA_ERR_INVALID_ARG;
    *fused = false;
    const Gate gate{g, nullptr, ld, m, nullptr, fused, keep_u};
    return guarded([&]() -> int {
        return group_fwd_checked(desc, X, A_all, B, Y, Z_all, H_all, ws, ws_bytes, stream, &gate);
    });
}

int layer_bwd_gated(const cola_desc* desc, const void* dY, const void* X, const void* Z, const void* H,
                    const void* A, const void* B, void* dX, float* dA, float* dB, void* ws, size_t ws_bytes,
                    cola_stream_t stream, const void* g, const void* u, int64_t ld, void* dg, void* du,
                    bool* fused) {
    if (!fused) return COLA_ERR_INVALID_ARG;
    *fused = false;
    const Gate gate{g, u, ld, dg, du, fused, true};
    return guarded([&]() -> int {
        return bwd_checked(desc, dY, X, Z, H, A, B, dX, dA, dB, ws, ws_bytes, stream, &gate);
    });
}

}  // namespace cola
