// gemm_skinny.hip -- the forward products of a few tokens (decode): C[M][N] =
// sum_k P(m, k) Q(n, k), M <= 64 token rows P, weight rows Q, both k-contiguous,
// fp32 accumulation, any alignment.
//
// What bounds it: each weight is used once, so the product streams Q; at the
// sizes of one projection that is latency, not bandwidth (one token of a 1B
// projection: 2 MB per product).  The 64 x 64 tiles ran K as a serial chain of
// K tiles on N / 64 workgroups (8 of them for Z of that projection: 9.4 us).
//  * A workgroup owns NB = 32 columns (16 for up to 32 tokens: twice the
//    workgroups, on the 16x16x32 instruction) and all tokens; its 8 waves take
//    every eighth 64-deep K tile each and add their sums in wave order at the end.
//  * Each wave moves its own K tiles: 16-byte element-aligned loads of whole
//    128-byte lines into registers, up to 8 K tiles ahead (what the registers
//    hold), so that a wave pays the memory latency once or twice in all, then
//    through a slice of LDS of its own into MFMA fragments.  No barriers until the
//    final sum.
// Kernel times, 64 x 64 tiles before -> these: one token of a 1B projection 14.3
// -> 8.6 us (both products); 32 tokens of 7B q, k and v 34 -> 17 us (50 MB of
// weights: 2.9 TB/s).  Two workgroups a CU (at most 128 registers a wave) beat
// twice the K tiles in flight: 17 against 20 us.
#include <type_traits>

#include "internal.hpp"
#include "device_math.hpp"

namespace cola {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NW = 8;
constexpr int NT = NW * 64;
constexpr int BK = 64;

struct SkinnyBatch {
    GemmArgs a[kMidBatch];
    int64_t first[kMidBatch + 1];
    int n;
};

// LDS offset of 16-byte chunk c of row r (128-byte rows, XOR swizzle: the rows
// of a fragment read cover the banks once)
__device__ __forceinline__ int off(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }

// R rows x 64 k of one operand in one wave's registers.
template <int R>
struct Rows {
    static constexpr int NI = R / 8;
    uint4 v[NI];
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
            v[i] = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
        }
    }
    __device__ __forceinline__ void put(char* lds, int lane) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) *reinterpret_cast<uint4*>(lds + off(8 * i + (lane >> 3), lane & 7)) = v[i];
    }
};

// Two consecutive columns gn, gn + 1 of row gm from their fp32 sums.
template <int EPI>
__device__ __forceinline__ void store2(const GemmArgs& a, int64_t gm, int64_t gn, float x0, float x1) {
    if (gm >= a.M || gn >= a.N) return;
    auto put = [&](void* base, int64_t ld, uint32_t w) {
        uint16_t* p = reinterpret_cast<uint16_t*>(base) + gm * ld + gn;
        if (gn + 1 < a.N) __builtin_memcpy(p, &w, 4);
        else p[0] = (uint16_t)(w & 0xffffu);
    };
    const uint32_t z = pack_bf16x2(x0, x1);
    if constexpr (EPI == EPI_STORE) {
        put(a.c, a.ldc, z);
    } else {
        const uint32_t h = pack_bf16x2(act_sigma<true>(a.act, __uint_as_float(z << 16)),
                                       act_sigma<true>(a.act, __uint_as_float(z & 0xffff0000u)));
        if constexpr (EPI == EPI_H) {
            put(a.c, a.ldc, h);
        } else {
            put(a.c, a.ldc, z);
            if (a.aux) put(a.aux, a.ldaux, h);
        }
    }
}

// RP token rows (16, 32 or 64), NB weight rows, AHEAD K tiles in flight.
template <int RP, int NB, int AHEAD, int EPI>
__global__ __launch_bounds__(NT, RP <= 32 ? 4 : 2) void gemm_skinny_kernel(const SkinnyBatch bt) {
    constexpr int MT = RP / NB;                               // NB x NB tiles
    constexpr int STAGE = (RP + NB) * 128;
    constexpr int RLD = NB + 4;
    constexpr int RED = NW * RP * RLD * 4;
    constexpr int SMEM = NW * STAGE > RED ? NW * STAGE : RED;
    __shared__ __attribute__((aligned(1024))) char smem[SMEM];
    int64_t b = blockIdx.x;
    int pi = 0;
    while (pi + 1 < bt.n && b >= bt.first[pi + 1]) ++pi;
    const GemmArgs& a = bt.a[pi];
    const int64_t n0 = (b - bt.first[pi]) * NB;
    const uint16_t* P = reinterpret_cast<const uint16_t*>(a.p);
    const uint16_t* Q = reinterpret_cast<const uint16_t*>(a.q);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* const ps = smem + wave * STAGE;
    char* const qs = ps + RP * 128;

    // sums of C^T tiles: lane l holds token l % NB, register v the column
    // NB = 32: 8 (v / 4) + 4 (l / 32) + v % 4; NB = 16: 4 (l / 16) + v
    constexpr int NV = NB == 32 ? 16 : 4;
    using Acc = std::conditional_t<NB == 32, f32x16, f32x4>;
    Acc acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i] = Acc{};

    // whole K tiles wave, wave + 8, ... are this wave's, and the partial last one
    // if its number falls there
    const int tiles = (int)(a.K / BK);
    const int cnt = tiles > wave ? (tiles - wave + NW - 1) / NW : 0;
    const uint16_t* const P0 = P + (int64_t)wave * BK;
    const uint16_t* const Q0 = Q + n0 * a.ldq + (int64_t)wave * BK;
    uint32_t op[Rows<RP>::NI], oq[Rows<NB>::NI];
    Rows<RP>::offsets(op, a.ldp, 0, a.M, lane);
    Rows<NB>::offsets(oq, a.ldq, n0, a.N, lane);
    Rows<RP> rp[AHEAD];
    Rows<NB> rq[AHEAD];
    auto load = [&](int u, int i) __attribute__((always_inline)) {
        rq[u].load(Q0 + (int64_t)i * (NW * BK), oq);
        rp[u].load(P0 + (int64_t)i * (NW * BK), op);
    };
    // one wave's LDS accesses execute in order: no barrier needed
    auto compute = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_wave_barrier();
        if constexpr (NB == 32) {
#pragma unroll
            for (int s = 0; s < BK / 16; ++s) {
                const int c = 2 * s + (lane >> 5);
                const bf16x8 q = *reinterpret_cast<const bf16x8*>(qs + off(lane & 31, c));
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const bf16x8 p = *reinterpret_cast<const bf16x8*>(ps + off(32 * m + (lane & 31), c));
                    acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q, p, acc[m], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int s = 0; s < BK / 32; ++s) {
                const int c = 4 * s + (lane >> 4);
                const bf16x8 q = *reinterpret_cast<const bf16x8*>(qs + off(lane & 15, c));
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const bf16x8 p = *reinterpret_cast<const bf16x8*>(ps + off(16 * m + (lane & 15), c));
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q, p, acc[m], 0, 0, 0);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
        if (u < cnt) load(u, u);
    for (int i0 = 0; i0 < cnt; i0 += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (i0 + u >= cnt) break;
            rp[u].put(ps, lane);
            rq[u].put(qs, lane);
            if (i0 + u + AHEAD < cnt) load(u, i0 + u + AHEAD);
            compute();
        }
    }
    if (tiles % NW == wave && (int64_t)tiles * BK < a.K) {
        const int valid = (int)(a.K - (int64_t)tiles * BK);
        rq[0].load_tail(Q + n0 * a.ldq + (int64_t)tiles * BK, oq, valid, lane);
        rp[0].load_tail(P + (int64_t)tiles * BK, op, valid, lane);
        rp[0].put(ps, lane);
        rq[0].put(qs, lane);
        compute();
    }
    __syncthreads();                                          // the tiles give way to the sums
    float* const red = reinterpret_cast<float*>(smem);        // [wave][token][RLD]
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        float* r = red + (wave * RP + NB * m + (lane & (NB - 1))) * RLD;
#pragma unroll
        for (int g = 0; g < NV / 4; ++g)
            *reinterpret_cast<f32x4*>(r + 8 * g + 4 * (lane / NB)) =
                f32x4{acc[m][4 * g], acc[m][4 * g + 1], acc[m][4 * g + 2], acc[m][4 * g + 3]};
    }
    __syncthreads();
    for (int id = threadIdx.x; id < RP * NB / 2; id += NT) {
        const int r = id / (NB / 2), c = 2 * (id % (NB / 2));
        if (r >= a.M) break;                                  // later ids are later rows
        float x0 = 0.0f, x1 = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float2 s = *reinterpret_cast<const float2*>(red + (w * RP + r) * RLD + c);
            x0 += s.x;
            x1 += s.y;
        }
        store2<EPI>(a, r, n0 + c, x0, x1);
    }
}

template <int RP, int NB, int AHEAD, int EPI>
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
    hipLaunchKernelGGL((gemm_skinny_kernel<RP, NB, AHEAD, EPI>), dim3((unsigned)blocks), dim3(NT), 0, s, bt);
    return hipGetLastError();
}

template <int EPI>
hipError_t launch_e(const GemmArgs* a, int n, hipStream_t s) {
    if (a[0].M <= 16) return launch_t<16, 16, 4, EPI>(a, n, s);
    if (a[0].M <= 32) return launch_t<32, 16, 3, EPI>(a, n, s);
    return launch_t<64, 32, 3, EPI>(a, n, s);
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
