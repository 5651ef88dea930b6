// gemm_skinny.hip -- the forward products of a few tokens (decode): C[M][N] =
// sum_k P(m, k) Q(n, k), M <= 32 token rows P, weight rows Q, both k-contiguous,
// fp32 accumulation, any alignment.
//
// What bounds it: each weight is used once, so the product streams Q; at the
// sizes of one projection that is latency, not bandwidth (one token of a 1B
// projection: 2 MB per product).  The 64 x 64 tiles ran K as a serial chain of
// loads on N / 64 workgroups (8 of them for Z of that projection: 9.4 us).
//  * A workgroup owns 16 columns and all tokens.  Eight waves load K tiles (64
//    deep), one each, by 16-byte element-aligned loads of whole 128-byte lines into
//    registers, up to four K tiles ahead, and put them into LDS in windows of four.
//  * The sums run over k in increasing order, as in the other kernel families, so
//    that a token's values do not depend on how many tokens share the call: a wave
//    of its own per 16 tokens multiplies one K tile after the other.  The chain of
//    16x16x32 MFMAs (16 clocks each) keeps pace with the windows' way through LDS
//    (256 clocks each way for 16 tokens); it lags behind the loads by two windows.
// Kernel times (Z and Y together), 64 x 64 tiles -> these: one token of a 1B
// projection 14.3 -> 9.4 us; 32 tokens of 7B q, k and v 34 -> 18.6 us.  (Eight
// chains over every eighth K tile, added at the end, took 8.0 and 16.2 us, but gave
// a token of a small call other bits than the same token of a larger one.)
#include "internal.hpp"
#include "device_math.hpp"
#include "lds_tile.hpp"

namespace cola {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int NL = 8;                                        // loading waves
constexpr int BK = 64;
constexpr int NB = 16;                                       // columns of a workgroup
constexpr int WT = 4;                                        // K tiles of a window
constexpr int NBUF = 3;                                      // windows in LDS
constexpr int DEPTH = 4;                                     // fragment reads in flight
static_assert(NL == 2 * WT, "windows alternate between two halves of the loading waves");

struct SkinnyBatch {
    GemmArgs a[kMidBatch];
    int64_t first[kMidBatch + 1];
    int n;
};

// LDS offset of 16-byte chunk c of row r (128-byte rows, XOR swizzle: the rows
// of a fragment read cover the banks once)
__device__ __forceinline__ int off(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }

// R rows of one operand's K tile in a wave's registers.
template <int R>
struct Rows {
    static constexpr int NI = R / 8;
    u32x4 v[NI];
    // Byte offsets of this lane's chunks from (first row, k0); rows past the last
    // re-read it (their sums are not stored).
    __device__ static __forceinline__ void offsets(uint32_t (&o)[NI], int64_t ld, int64_t row0, int64_t rows, int lane) {
        const int64_t lim64 = rows - 1 - row0;
        const int lim = lim64 < R - 1 ? (int)lim64 : R - 1;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int r = 8 * i + (lane >> 3);
            o[i] = 2u * (uint32_t)(r < lim ? r : lim) * (uint32_t)ld + 16u * (uint32_t)(lane & 7);
        }
    }
    // a whole K tile: base is the first row's element at the tile's first k
    __device__ __forceinline__ void load(const uint16_t* base, const uint32_t (&o)[NI]) {
#pragma unroll
        for (int i = 0; i < NI; ++i) __builtin_memcpy(&v[i], reinterpret_cast<const char*>(base) + o[i], 16);
    }
    // the last, partial one: `valid` k from base on, then zeros
    __device__ __forceinline__ void load_tail(const uint16_t* base, const uint32_t (&o)[NI], int valid, int lane) {
        const int n = valid - 8 * (lane & 7);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            uint32_t e[8];
            const uint16_t* p = reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(base) + o[i]);
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = u < n ? (uint32_t)p[u] : 0u;
            v[i] = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
        }
    }
    __device__ __forceinline__ void put(char* lds, int lane) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) *reinterpret_cast<u32x4*>(lds + off(8 * i + (lane >> 3), lane & 7)) = v[i];
    }
};

// Four consecutive columns gn .. gn + 3 of row gm from their fp32 sums.
template <int EPI>
__device__ __forceinline__ void store4(const GemmArgs& a, int64_t gm, int64_t gn, f32x4 x) {
    if (gm >= a.M || gn >= a.N) return;
    const int n = (int)(a.N - gn < 4 ? a.N - gn : 4);
    auto put = [&](void* base, int64_t ld, uint32_t w0, uint32_t w1) {
        uint16_t* p = reinterpret_cast<uint16_t*>(base) + gm * ld + gn;
        if (n == 4) {
            const uint2 w = make_uint2(w0, w1);
            __builtin_memcpy(p, &w, 8);
        } else {
            p[0] = (uint16_t)(w0 & 0xffffu);
            if (n > 1) p[1] = (uint16_t)(w0 >> 16);
            if (n > 2) p[2] = (uint16_t)(w1 & 0xffffu);
        }
    };
    const uint32_t z0 = pack_bf16x2(x[0], x[1]), z1 = pack_bf16x2(x[2], x[3]);
    if constexpr (EPI == EPI_STORE) {
        put(a.c, a.ldc, z0, z1);
    } else {
        auto sigma = [&](uint32_t z) {
            return pack_bf16x2(act_sigma<true>(a.act, __uint_as_float(z << 16)),
                               act_sigma<true>(a.act, __uint_as_float(z & 0xffff0000u)));
        };
        const uint32_t h0 = sigma(z0), h1 = sigma(z1);
        if constexpr (EPI == EPI_H) {
            put(a.c, a.ldc, h0, h1);
        } else {
            put(a.c, a.ldc, z0, z1);
            if (a.aux) put(a.aux, a.ldaux, h0, h1);
        }
    }
}

// RP token rows (16 or 32): one multiplying wave for every 16 of them.
template <int RP>
struct Geo {
    static constexpr int THREADS = 64 * (NL + RP / 16);
    static constexpr int TILE = (RP + NB) * 128;              // one K tile: the token rows, then the weight rows
    static constexpr int WINDOW = WT * TILE;
    static_assert(2 * NBUF * WINDOW <= 160 * 1024, "two workgroups a CU");
};

// AHEAD: K tiles that a loading wave has in flight.
template <int RP, int AHEAD, int EPI>
__global__ __launch_bounds__(Geo<RP>::THREADS, 5) void gemm_skinny_kernel(const SkinnyBatch bt) {
    using G = Geo<RP>;
    __shared__ __attribute__((aligned(1024))) char smem[NBUF * G::WINDOW];
    int64_t b = blockIdx.x;
    int pi = 0;
    while (pi + 1 < bt.n && b >= bt.first[pi + 1]) ++pi;
    const GemmArgs& a = bt.a[pi];
    const int64_t n0 = (b - bt.first[pi]) * NB;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // Window i, in buffer i % 3, holds the whole K tiles 4 i .. 4 i + 3, loaded by
    // waves 0 .. 3 (even i) or 4 .. 7 (odd).  Barrier i says that window i is in
    // place; a multiplying wave passes it before it works on window i - 1 (whose last
    // steps read ahead into window i), so it has left window i - 2 by then and buffer
    // (i + 1) % 3 may be filled.  The partial last K tile is a window of its own.
    const int tiles = (int)(a.K / BK);
    const int windows = (tiles + WT - 1) / WT;
    const int64_t kt = (int64_t)tiles * BK;
    const bool tail = kt < a.K;
    if (wave < NL) {
        const uint16_t* const P = reinterpret_cast<const uint16_t*>(a.p);
        const uint16_t* const Q = reinterpret_cast<const uint16_t*>(a.q) + n0 * a.ldq;
        uint32_t op[Rows<RP>::NI], oq[Rows<NB>::NI];
        Rows<RP>::offsets(op, a.ldp, 0, a.M, lane);
        Rows<NB>::offsets(oq, a.ldq, n0, a.N, lane);
        if (tiles > 0) {
            const int odd = wave / WT;
            const int pairs = (windows + 1) / 2;              // window 2 j + odd is this wave's
            Rows<RP> p[AHEAD];
            Rows<NB> q[AHEAD];
            // Past the last whole K tile it is read again and not used: with a branch
            // around the loads, or their order not fixed, the waits before a put would
            // be for all of them.
            auto load = [&](int u, int j) __attribute__((always_inline)) {
                const int t = 2 * WT * j + wave < tiles ? 2 * WT * j + wave : tiles - 1;
                q[u].load(Q + (int64_t)t * BK, oq);
                p[u].load(P + (int64_t)t * BK, op);
                __builtin_amdgcn_sched_barrier(0);
            };
            auto put = [&](int u, int j) __attribute__((always_inline)) {
                char* const d = smem + (2 * j + odd) % NBUF * G::WINDOW + wave % WT * G::TILE;
                q[u].put(d + RP * 128, lane);
                p[u].put(d, lane);
                __builtin_amdgcn_sched_barrier(0);
            };
            static_for<AHEAD>([&](auto u) __attribute__((always_inline)) { load(u, u); });
            int j0 = 0;
            for (; j0 + AHEAD < pairs; j0 += AHEAD)
                static_for<AHEAD>([&](auto u) __attribute__((always_inline)) {
                    if (odd) __syncthreads();
                    put(u, j0 + u);
                    load(u, j0 + u + AHEAD);
                    __syncthreads();
                    if (!odd) __syncthreads();
                });
            static_for<AHEAD>([&](auto u) __attribute__((always_inline)) {
                if (j0 + u < pairs) {
                    const bool two = 2 * (j0 + u) + 1 < windows;
                    if (odd) __syncthreads();
                    if (two || !odd) {
                        put(u, j0 + u);
                        __syncthreads();
                    }
                    if (two && !odd) __syncthreads();
                }
            });
        }
        if (tail) {
            if (wave == 0) {
                char* const d = smem + windows % NBUF * G::WINDOW;
                Rows<RP> p;
                Rows<NB> q;
                q.load_tail(Q + kt, oq, (int)(a.K - kt), lane);
                p.load_tail(P + kt, op, (int)(a.K - kt), lane);
                q.put(d + RP * 128, lane);
                p.put(d, lane);
            }
            __syncthreads();
        }
        return;
    }

    // sums of a C^T tile: lane l holds token l % 16 of the wave's, columns
    // 4 (l / 16) + 0..3
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    const int m0 = 16 * (wave - NL);
    constexpr int SPT = BK / 32;                              // steps of a K tile
    constexpr int SPW = WT * SPT;
    const int o[SPT] = {off(lane & 15, lane >> 4), off(lane & 15, 4 + (lane >> 4))};
    struct Frag {
        bf16x8 q, p;
    };
    auto read = [&](const char* st, int s) __attribute__((always_inline)) {
        const char* const t = st + s / SPT * G::TILE + o[s % SPT];
        return Frag{*reinterpret_cast<const bf16x8*>(t + RP * 128), *reinterpret_cast<const bf16x8*>(t + m0 * 128)};
    };
    auto mfma = [&](const Frag& f) __attribute__((always_inline)) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.q, f.p, acc, 0, 0, 0);
    };
    if (tiles > 0) {
        Frag f[DEPTH];
        __syncthreads();
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) f[s] = read(smem, s);
        int cur = 0;
        for (int i = 0; i + 1 < windows; ++i) {
            __syncthreads();
            const int nxt = cur + 1 == NBUF ? 0 : cur + 1;
            const char *const c = smem + cur * G::WINDOW, *const n = smem + nxt * G::WINDOW;
#pragma unroll
            for (int s = 0; s < SPW; ++s) {
                __builtin_amdgcn_sched_barrier(0);
                mfma(f[s % DEPTH]);
                f[s % DEPTH] = s + DEPTH < SPW ? read(c, s + DEPTH) : read(n, s + DEPTH - SPW);
            }
            cur = nxt;
        }
        const char* const c = smem + cur * G::WINDOW;
        const int left = SPT * (tiles - WT * (windows - 1));  // steps of the last window
#pragma unroll
        for (int s = 0; s < SPW; ++s) {
            if (s < left) {
                mfma(f[s % DEPTH]);
                if (s + DEPTH < SPW) f[s % DEPTH] = read(c, s + DEPTH);
            }
        }
    }
    if (tail) {
        __syncthreads();
        const char* const c = smem + windows % NBUF * G::WINDOW;
#pragma unroll
        for (int s = 0; s < SPT; ++s) mfma(read(c, s));
    }
    store4<EPI>(a, m0 + (lane & 15), n0 + 4 * (lane >> 4), acc);
}

template <int RP, int AHEAD, int EPI>
hipError_t launch_t(const GemmArgs* a, int n, hipStream_t s) {
    SkinnyBatch bt;
    bt.n = n;
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        if (a[i].p_layout != KMAJ || a[i].q_layout != KMAJ || a[i].epi != EPI || a[i].M != a[0].M || a[i].splits != 1)
            return hipErrorInvalidValue;
        bt.a[i] = a[i];
        bt.first[i] = blocks;
        blocks += (a[i].N + NB - 1) / NB;
    }
    for (int i = n; i <= kMidBatch; ++i) bt.first[i] = blocks;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_skinny_kernel<RP, AHEAD, EPI>), dim3((unsigned)blocks), dim3(Geo<RP>::THREADS), 0, s, bt);
    return hipGetLastError();
}

// K tiles in flight: what the registers hold, or fewer where K has no more (loads past
// the end would only be in the way).
template <int RP, int EPI>
hipError_t launch_k(const GemmArgs* a, int n, hipStream_t s) {
    int64_t K = 0;
    for (int i = 0; i < n; ++i) K = a[i].K > K ? a[i].K : K;
    if (K <= NL * BK) return launch_t<RP, 1, EPI>(a, n, s);
    if (K <= 2 * NL * BK) return launch_t<RP, 2, EPI>(a, n, s);
    return launch_t<RP, RP == 16 ? 4 : 3, EPI>(a, n, s);
}

template <int EPI>
hipError_t launch_e(const GemmArgs* a, int n, hipStream_t s) {
    return a[0].M <= 16 ? launch_k<16, EPI>(a, n, s) : launch_k<32, EPI>(a, n, s);
}

}  // namespace

hipError_t launch_gemm_skinny(const GemmArgs* a, int n, hipStream_t s) {
    if (n < 1 || n > kMidBatch || a[0].M < 1 || a[0].M > kSkinnyRows) return hipErrorInvalidValue;
    switch (a[0].epi) {
        case EPI_STORE: return launch_e<EPI_STORE>(a, n, s);
        case EPI_H: return launch_e<EPI_H>(a, n, s);
        case EPI_Z_H: return launch_e<EPI_Z_H>(a, n, s);
        default: return hipErrorNotSupported;
    }
}

}  // namespace cola
