// gemm_f32.hip -- fp32 storage path: C[M][N] = sum_k P(m, k) Q(n, k) on the
// fp32 matrix instruction (v_mfma_f32_32x32x2_f32: fp32 products and sums, no
// reduced-precision shortcut), the same operand layouts and epilogues as the
// bf16 kernels; any shape, pitch and 4-byte alignment.
//
// What bounds it: the products of this path are small (a few hundred to a few
// thousand rows), so a launch is a chain of latencies on a mostly idle chip;
// 32-deep K tiles go global -> registers (one tile ahead) -> LDS -> fragments.
//  * narrow: 32 x 32 output tiles; the eight waves of a workgroup take every
//    eighth K tile each, through LDS of their own (no barriers in the K loop),
//    and their sums are added in wave order at the end.  Fills the chip from
//    256 tiles of 32 x 32 on and shortens the K chain eightfold.
//  * wide: 64 x 64 tiles, each wave a 32 x 32 quarter over all of K, operands
//    shared through double-buffered LDS: half the traffic per flop.  Used once
//    256 such tiles (or splits of them) exist.
// A training step of T = 256, 512 -> 128 -> 512 takes 24 us, bound by its four
// launches; a 64 x 64 VALU kernel took 213 (8 workgroups and 50 us for Z alone).
// A value's last bits depend on the variant, and so on how many tokens share the
// call: either order of the sum is within the fp32 rounding of the other.
// LDS: k-contiguous operands as [row][32 k] with rows of 36 floats, m-contiguous
// ones as [k][rows] with rows of rows + 8 floats: the 16-byte fragment reads of
// the former and the two 4-byte half-wave rows (4 k apart) of the latter fall
// into distinct banks.
#include "internal.hpp"
#include "device_math.hpp"

namespace cola {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int BK = F32_BK;
static_assert(BK == 32, "K tile of 8 four-float chunks");

// Operand tile of R rows x 32 k, moved by NT threads (16 bytes each at a time).
template <int LAYOUT, int R, int NT>
struct FTile {
    static constexpr int LD = LAYOUT == KMAJ ? BK + 4 : R + 8;        // floats per LDS row
    static constexpr int FLOATS = LAYOUT == KMAJ ? R * LD : BK * LD;
    static constexpr int CPR = LAYOUT == KMAJ ? BK / 4 : R / 4;       // chunks per LDS row
    static constexpr int NI = R * BK / 4 / NT;
    f32x4_t v[NI];

    // rows row0 .., k from k0; zeros past the edges
    __device__ __forceinline__ void load(const float* base, int64_t ld, int64_t row0, int64_t rows, int64_t k0,
                                         int64_t kend, int t) {
        // whole tiles (a uniform condition): every load in flight at once (guarded
        // one by one they wait for each other)
        if (row0 + R <= rows && k0 + BK <= kend) {
            const float* p = LAYOUT == KMAJ ? base + row0 * ld + k0 : base + k0 * ld + row0;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int id = t + NT * i;
                __builtin_memcpy(&v[i], p + (int64_t)(id / CPR) * ld + 4 * (id % CPR), 16);   // 4-byte alignment is enough
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int id = t + NT * i;
            const int a = id / CPR, c = 4 * (id % CPR);
            // a: row (k-contiguous) or k; c: first k or first row of the chunk
            const int64_t o = LAYOUT == KMAJ ? row0 + a : k0 + a, olim = LAYOUT == KMAJ ? rows : kend;
            const int64_t e = LAYOUT == KMAJ ? k0 + c : row0 + c, elim = LAYOUT == KMAJ ? kend : rows;
            f32x4_t x = {0.0f, 0.0f, 0.0f, 0.0f};
            if (o < olim) {
                const float* p = base + o * ld + e;
                if (e + 4 <= elim) {
                    __builtin_memcpy(&x, p, 16);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (e + u < elim) x[u] = p[u];
                }
            }
            v[i] = x;
        }
    }
    __device__ __forceinline__ void put(float* lds, int t) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int id = t + NT * i;
            *reinterpret_cast<f32x4_t*>(lds + (id / CPR) * LD + 4 * (id % CPR)) = v[i];
        }
    }
    // the four matrix steps of k group j (k = 8 j + 4 (lane / 32) + 0..3) of rows
    // r0 .. r0 + 31
    __device__ static __forceinline__ f32x4_t frag(const float* lds, int r0, int j, int lane) {
        const int r = r0 + (lane & 31), k = 8 * j + 4 * (lane >> 5);
        if constexpr (LAYOUT == KMAJ) {
            return *reinterpret_cast<const f32x4_t*>(lds + r * LD + k);
        } else {
            f32x4_t x;
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = lds[(k + u) * LD + r];
            return x;
        }
    }
};

// Epilogue of 4 consecutive columns gn .. gn + 3 of row gm.
template <int EPI>
__device__ __forceinline__ void epilogue(const GemmArgs& a, int split, int64_t gm, int64_t gn, f32x4_t x) {
    if (gm >= a.M || gn >= a.N) return;
    const int n = (int)(a.N - gn < 4 ? a.N - gn : 4);
    auto store = [n](float* p, f32x4_t y) {
        if (n == 4) {
            __builtin_memcpy(p, &y, 16);
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (e < n) p[e] = y[e];
        }
    };
    float* c = reinterpret_cast<float*>(a.c) + (int64_t)split * a.split_stride + gm * a.ldc + gn;
    float* h = a.aux ? reinterpret_cast<float*>(a.aux) + gm * a.ldaux + gn : nullptr;
    f32x4_t y = x, s = x;
    if constexpr (EPI == EPI_Z_H || EPI == EPI_H) {
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = act_sigma<false>(a.act, x[e]);
        if (EPI == EPI_H) y = s;
    } else if constexpr (EPI == EPI_DZ) {
        const float* zp = reinterpret_cast<const float*>(a.zin) + gm * a.ldzin + gn;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float z = e < n ? zp[e] : 0.0f;
            y[e] = x[e] * act_sigma_prime<false>(a.act, z);
            if (h) s[e] = act_sigma<false>(a.act, z);
        }
    }
    store(c, y);
    if constexpr (EPI == EPI_Z_H || EPI == EPI_DZ) {
        if (h) store(h, s);
    }
}

struct F32Batch {
    GemmArgs a[kF32Batch];
    int64_t first[kF32Batch + 1];
    int n;
};

// acc (C^T: lane l holds row l % 32, registers 4 g .. 4 g + 3 the columns
// 8 g + 4 (l / 32) + 0..3) += the 32 x 32 products of one K tile
template <class TP, class TQ>
__device__ __forceinline__ void mfma_tile(f32x16_t& acc, const float* ps, const float* qs, int rp, int rq, int lane) {
#pragma unroll
    for (int j = 0; j < BK / 8; ++j) {
        const f32x4_t p = TP::frag(ps, rp, j, lane), q = TQ::frag(qs, rq, j, lane);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(q[u], p[u], acc, 0, 0, 0);
    }
}

constexpr int NWK = 8;                                                // waves that share K (narrow)

// LDS floats of a workgroup; narrow: also room for the waves' sums,
// [wave][32][RLD].
constexpr int RLD = 36;
template <int PL, int QL, bool WIDE>
constexpr int f32_smem() {
    constexpr int TB = WIDE ? 64 : 32, NT = WIDE ? 256 : 64;
    constexpr int tiles = (WIDE ? 2 : NWK) * (FTile<PL, TB, NT>::FLOATS + FTile<QL, TB, NT>::FLOATS);
    return WIDE || tiles > NWK * 32 * RLD ? tiles : NWK * 32 * RLD;
}

// This block's product, and its number within it.
__device__ __forceinline__ uint32_t f32_block(const F32Batch& bt, int* product) {
    int pi = 0;
    while (pi + 1 < bt.n && (int64_t)blockIdx.x >= bt.first[pi + 1]) ++pi;
    *product = pi;
    return blockIdx.x - (uint32_t)bt.first[pi];                       // fewer than 2^31 blocks
}

// Output tile (and split) number b of the product a.
template <int PL, int QL, int EPI, bool WIDE>
__device__ __forceinline__ void f32_tile(const GemmArgs& a, uint32_t b, float* smem) {
    constexpr int TB = WIDE ? 64 : 32;
    constexpr int NT = WIDE ? 256 : 64;                               // threads that share an LDS tile
    using TP = FTile<PL, TB, NT>;
    using TQ = FTile<QL, TB, NT>;
    constexpr int STAGE = TP::FLOATS + TQ::FLOATS;
    const uint32_t tiles_n = (uint32_t)((a.N + TB - 1) / TB);
    const uint32_t per_split = tiles_n * (uint32_t)((a.M + TB - 1) / TB);
    int split = 0;
    if (a.splits > 1) {
        split = (int)(b / per_split);
        b -= (uint32_t)split * per_split;
    }
    const uint32_t tm = b / tiles_n;
    const int64_t m0 = (int64_t)tm * TB, n0 = (int64_t)(b - tm * tiles_n) * TB;
    const int64_t kbeg = (int64_t)split * a.k_chunk;
    const int64_t kend = min(a.K, kbeg + a.k_chunk);
    const float* P = reinterpret_cast<const float*>(a.p);
    const float* Q = reinterpret_cast<const float*>(a.q);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    TP tp;
    TQ tq;
    if constexpr (WIDE) {
        const int t = threadIdx.x;
        tp.load(P, a.ldp, m0, a.M, kbeg, kend, t);
        tq.load(Q, a.ldq, n0, a.N, kbeg, kend, t);
        int buf = 0;
        for (int64_t k0 = kbeg; k0 < kend; k0 += BK, buf ^= 1) {
            // a wave writes the buffer of two K tiles ago: every wave has left
            // it, since it passed the barrier of the K tile in between
            float* s = smem + buf * STAGE;
            tp.put(s, t);
            tq.put(s + TP::FLOATS, t);
            __syncthreads();
            if (k0 + BK < kend) {
                tp.load(P, a.ldp, m0, a.M, k0 + BK, kend, t);
                tq.load(Q, a.ldq, n0, a.N, k0 + BK, kend, t);
            }
            mfma_tile<TP, TQ>(acc, s, s + TP::FLOATS, 32 * (wave >> 1), 32 * (wave & 1), lane);
        }
        const int64_t gm = m0 + 32 * (wave >> 1) + (lane & 31);
#pragma unroll
        for (int g = 0; g < 4; ++g)
            epilogue<EPI>(a, split, gm, n0 + 32 * (wave & 1) + 8 * g + 4 * (lane >> 5),
                          f32x4_t{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]});
    } else {
        float* s = smem + wave * STAGE;                               // this wave's own
        int64_t k0 = kbeg + wave * BK;
        tp.load(P, a.ldp, m0, a.M, k0, kend, lane);
        tq.load(Q, a.ldq, n0, a.N, k0, kend, lane);
        for (; k0 < kend; k0 += NWK * BK) {
            // one wave's LDS accesses execute in order: no barrier needed
            tp.put(s, lane);
            tq.put(s + TP::FLOATS, lane);
            if (k0 + NWK * BK < kend) {
                tp.load(P, a.ldp, m0, a.M, k0 + NWK * BK, kend, lane);
                tq.load(Q, a.ldq, n0, a.N, k0 + NWK * BK, kend, lane);
            }
            __builtin_amdgcn_wave_barrier();
            mfma_tile<TP, TQ>(acc, s, s + TP::FLOATS, 0, 0, lane);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();                                              // the tiles give way to the sums
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4_t*>(smem + (32 * wave + (lane & 31)) * RLD + 8 * g + 4 * (lane >> 5)) =
                f32x4_t{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
        __syncthreads();
        if (threadIdx.x >= 256) return;
        const int r = threadIdx.x >> 3, c = 4 * (threadIdx.x & 7);
        f32x4_t x = *reinterpret_cast<const f32x4_t*>(smem + r * RLD + c);
#pragma unroll
        for (int w = 1; w < NWK; ++w) x += *reinterpret_cast<const f32x4_t*>(smem + (32 * w + r) * RLD + c);
        epilogue<EPI>(a, split, m0 + r, n0 + c, x);
    }
}

template <int PL, int QL, int EPI, bool WIDE>
__global__ __launch_bounds__(WIDE ? 256 : 64 * NWK) void gemm_f32_kernel(const F32Batch bt) {
    __shared__ __attribute__((aligned(16))) float smem[f32_smem<PL, QL, WIDE>()];
    int pi;
    const uint32_t b = f32_block(bt, &pi);
    f32_tile<PL, QL, EPI, WIDE>(bt.a[pi], b, smem);
}

// dX = dZ A (product 0) and the weight gradients (the rest), which both follow
// from dZ, in one grid.
__global__ __launch_bounds__(64 * NWK) void gemm_f32_dxw_kernel(const F32Batch bt) {
    constexpr int S0 = f32_smem<KMAJ, MNMAJ, false>(), S1 = f32_smem<MNMAJ, MNMAJ, false>();
    __shared__ __attribute__((aligned(16))) float smem[S0 > S1 ? S0 : S1];
    int pi;
    const uint32_t b = f32_block(bt, &pi);
    if (pi == 0) f32_tile<KMAJ, MNMAJ, EPI_STORE, false>(bt.a[0], b, smem);
    else f32_tile<MNMAJ, MNMAJ, EPI_STORE_F32, false>(bt.a[pi], b, smem);
}

bool f32_wide(const GemmArgs* a, int n) {
    int64_t t64 = 0;
    for (int i = 0; i < n; ++i) t64 += f32_tiles(64, a[i].M, a[i].N) * a[i].splits;
    return t64 >= 256;
}

template <int PL, int QL, int EPI>
hipError_t launch_t(const GemmArgs* a, int n, hipStream_t s) {
    for (int i = 0; i < n; ++i)
        if (a[i].p_layout != PL || a[i].q_layout != QL || a[i].epi != EPI) return hipErrorInvalidValue;
    const bool wide = f32_wide(a, n);
    F32Batch bt;
    bt.n = n;
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        bt.a[i] = a[i];
        bt.first[i] = blocks;
        blocks += f32_tiles(wide ? 64 : 32, a[i].M, a[i].N) * a[i].splits;
    }
    for (int i = n; i <= kF32Batch; ++i) bt.first[i] = blocks;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if (wide) hipLaunchKernelGGL((gemm_f32_kernel<PL, QL, EPI, true>), dim3((unsigned)blocks), dim3(256), 0, s, bt);
    else hipLaunchKernelGGL((gemm_f32_kernel<PL, QL, EPI, false>), dim3((unsigned)blocks), dim3(64 * NWK), 0, s, bt);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_f32_batch(const GemmArgs* a, int n, hipStream_t s) {
    if (n < 1 || n > kF32Batch) return hipErrorInvalidValue;
    const int pl = a[0].p_layout, ql = a[0].q_layout;
    switch (a[0].epi) {
        case EPI_Z_H:
            if (pl == KMAJ && ql == KMAJ) return launch_t<KMAJ, KMAJ, EPI_Z_H>(a, n, s);
            break;
        case EPI_H:
            if (pl == KMAJ && ql == KMAJ) return launch_t<KMAJ, KMAJ, EPI_H>(a, n, s);
            break;
        case EPI_STORE:
            if (pl == KMAJ && ql == KMAJ) return launch_t<KMAJ, KMAJ, EPI_STORE>(a, n, s);
            if (pl == KMAJ && ql == MNMAJ) return launch_t<KMAJ, MNMAJ, EPI_STORE>(a, n, s);
            break;
        case EPI_DZ:
            if (pl == KMAJ && ql == MNMAJ) return launch_t<KMAJ, MNMAJ, EPI_DZ>(a, n, s);
            break;
        case EPI_STORE_F32:
            if (pl == MNMAJ && ql == MNMAJ) return launch_t<MNMAJ, MNMAJ, EPI_STORE_F32>(a, n, s);
            break;
        default:
            break;
    }
    return hipErrorNotSupported;
}

bool f32_dxw_takes(const GemmArgs* a, int n) { return n <= kF32Batch && !f32_wide(a, 1) && !f32_wide(a + 1, n - 1); }

hipError_t launch_gemm_f32_dxw(const GemmArgs* a, int n, hipStream_t s) {
    if (n < 2 || n > kF32Batch) return hipErrorInvalidValue;
    F32Batch bt;
    bt.n = n;
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        if (a[i].p_layout != (i == 0 ? KMAJ : MNMAJ) || a[i].q_layout != MNMAJ ||
            a[i].epi != (i == 0 ? EPI_STORE : EPI_STORE_F32))
            return hipErrorInvalidValue;
        bt.a[i] = a[i];
        bt.first[i] = blocks;
        blocks += f32_tiles(32, a[i].M, a[i].N) * a[i].splits;
    }
    for (int i = n; i <= kF32Batch; ++i) bt.first[i] = blocks;
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(gemm_f32_dxw_kernel, dim3((unsigned)blocks), dim3(64 * NWK), 0, s, bt);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// split-K reduction, zero fill, and row repacking of 16-bit weights
// ---------------------------------------------------------------------------
namespace {

// The split reduction's fixed order, which depends only on the split count:
// the partials in chunks of kChunk in split order, each chunk summed in
// order, then the chunk sums in order (up to kChunk splits: the plain sum in
// split order).  Two kernels follow it: one thread per output group summing
// every chunk in turn, and, for split counts above kChunk, kChunkLanes
// threads per output group summing chunks side by side and combining them in
// LDS, which keeps several times as many loads in flight when the output is
// small.
constexpr int kChunk = 8;
constexpr int kChunkLanes = 4;
constexpr int kMaxChunks = 32;

__device__ __forceinline__ float4 add4(float4 a, float4 b) {
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}
__device__ __forceinline__ float add4(float a, float b) { return a + b; }

// Sum of partials k0 .. k1-1 (k1 > k0) of element i; V = float4 (stride in
// float4 units) or float.
// (All of a chunk's loads are issued before its sums.)
template <class V>
__device__ __forceinline__ V chunk_sum(const V* __restrict__ part, int64_t stride, int64_t i, int k0, int k1) {
    V v[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u)
        if (k0 + u < k1) v[u] = part[(int64_t)(k0 + u) * stride + i];
    V s = v[0];
#pragma unroll
    for (int u = 1; u < kChunk; ++u)
        if (k0 + u < k1) s = add4(s, v[u]);
    return s;
}

template <class V>
__device__ __forceinline__ V ordered_sum(const V* __restrict__ part, int64_t stride, int64_t i, int splits) {
    V s = chunk_sum(part, stride, i, 0, min(kChunk, splits));
    for (int k0 = kChunk; k0 < splits; k0 += kChunk) s = add4(s, chunk_sum(part, stride, i, k0, min(k0 + kChunk, splits)));
    return s;
}

bool reduce_vec_ok(const float* part, int64_t stride, const float* out) {
    return (stride & 3) == 0 && (reinterpret_cast<uintptr_t>(part) & 15u) == 0 &&
           (reinterpret_cast<uintptr_t>(out) & 15u) == 0;
}

// One thread per output group, block blk of nblk (grid-stride over float4
// groups, scalar tail).
__device__ __forceinline__ void reduce_splits_range(const float* __restrict__ part, int splits, int64_t stride,
                                                    float* __restrict__ out, int64_t n, int64_t blk,
                                                    int64_t nblk) {
    const int64_t n4 = n >> 2;
    const bool vec = ((stride & 3) == 0) && ((reinterpret_cast<uintptr_t>(part) & 15u) == 0) &&
                     ((reinterpret_cast<uintptr_t>(out) & 15u) == 0);
    const int64_t step = nblk * blockDim.x;
    int64_t i = blk * blockDim.x + threadIdx.x;
    if (vec) {
        const float4* p4 = reinterpret_cast<const float4*>(part);
        for (; i < n4; i += step) reinterpret_cast<float4*>(out)[i] = ordered_sum(p4, stride >> 2, i, splits);
        // scalar tail
        i = n4 * 4 + blk * blockDim.x + threadIdx.x;
    }
    for (; i < n; i += step) out[i] = ordered_sum(part, stride, i, splits);
}

// kChunkLanes threads per float4 output group (n a multiple of 4, 16-byte
// aligned rows): 256 / kChunkLanes groups per block.
__device__ __forceinline__ void reduce_chunks_range(const float* __restrict__ part, int splits, int64_t stride,
                                                    float* __restrict__ out, int64_t n, int64_t blk) {
    constexpr int OPB = 256 / kChunkLanes;
    __shared__ float4 sums[kMaxChunks][OPB];
    const int j = threadIdx.x / OPB, o = threadIdx.x % OPB;
    const int64_t i = blk * OPB + o, n4 = n >> 2;
    const int chunks = (splits + kChunk - 1) / kChunk;
    const float4* p4 = reinterpret_cast<const float4*>(part);
    if (i < n4)
        for (int c = j; c < chunks; c += kChunkLanes)
            sums[c][o] = chunk_sum(p4, stride >> 2, i, kChunk * c, min(kChunk * c + kChunk, splits));
    __syncthreads();
    if (j == 0 && i < n4) {
        float4 s = sums[0][o];
        for (int c = 1; c < chunks; ++c) s = add4(s, sums[c][o]);
        reinterpret_cast<float4*>(out)[i] = s;
    }
}

// Up to kReduceBatch reductions with one split count in a launch: blocks
// [first[i], first[i + 1]) sum the partials of job i (the order does not depend on
// what shares the launch).
struct ReduceBatch {
    ReduceJob j[kReduceBatch];
    int64_t first[kReduceBatch + 1];
    int n, splits;
};

template <bool CHUNKS>
__global__ __launch_bounds__(256) void reduce_kernel(const ReduceBatch bt) {
    const int64_t b = blockIdx.x;
    int i = 0;
    while (i + 1 < bt.n && b >= bt.first[i + 1]) ++i;
    const ReduceJob& r = bt.j[i];
    if constexpr (CHUNKS) reduce_chunks_range(r.part, bt.splits, r.n, r.out, r.n, b - bt.first[i]);
    else reduce_splits_range(r.part, bt.splits, r.n, r.out, r.n, b - bt.first[i], bt.first[i + 1] - bt.first[i]);
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float* __restrict__ out, int64_t n) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) out[i] = 0.0f;
}

// dst[r][c] = src[r][c], c < width, 0 up to ld: rows of 16-byte chunks, 1 << shift
// threads a row (a power of two near the chunk count), whole chunks read with one
// element-aligned 16-byte load.
__global__ __launch_bounds__(256) void pack_rows_kernel(const uint16_t* __restrict__ src, int64_t src_ld,
                                                        int64_t rows, int64_t width, uint16_t* __restrict__ dst,
                                                        int64_t ld, int shift) {
    const int per = 256 >> shift;                            // rows a block takes at a time
    const int t = threadIdx.x & ((1 << shift) - 1);
    const int64_t chunks = ld >> 3;
    for (int64_t r = (int64_t)blockIdx.x * per + (threadIdx.x >> shift); r < rows; r += (int64_t)gridDim.x * per) {
        const uint16_t* s = src + r * src_ld;
        uint16_t* d = dst + r * ld;
        for (int64_t c = t; c < chunks; c += 1 << shift) {
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (8 * c + 8 <= width) {
                __builtin_memcpy(&v, s + 8 * c, 16);
            } else {
                uint32_t e[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) e[k] = 8 * c + k < width ? (uint32_t)s[8 * c + k] : 0u;
                v = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
            }
            *reinterpret_cast<uint4*>(d + 8 * c) = v;
        }
    }
}

// dP = dY (.) sigma'(P) (the both-sigma variant's backward through its outer
// sigma).  One thread per group of V consecutive elements of a row (V = 8 for
// bf16, 4 for fp32: one 16-byte access per operand when every row start is
// 16-byte aligned), grid-stride over the groups.  bf16 products are taken in
// fp32 and rounded to nearest even.
template <bool BF16>
__global__ __launch_bounds__(256) void outer_grad_kernel(const void* __restrict__ dy, int64_t lddy,
                                                         const void* __restrict__ p, int64_t ldp,
                                                         void* __restrict__ out, int64_t ldo, int64_t T,
                                                         int64_t n, int act, int vec) {
    constexpr int V = BF16 ? 8 : 4;
    const int64_t groups = (n + V - 1) / V;
    const int64_t total = T * groups;
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += step) {
        const int64_t t = g / groups;
        const int64_t c0 = (g - t * groups) * V;
        const int valid = (int)(n - c0 < V ? n - c0 : V);
        if constexpr (BF16) {
            const uint16_t* a = reinterpret_cast<const uint16_t*>(dy) + t * lddy + c0;
            const uint16_t* b = reinterpret_cast<const uint16_t*>(p) + t * ldp + c0;
            uint16_t* o = reinterpret_cast<uint16_t*>(out) + t * ldo + c0;
            if (vec && valid == V) {
                const uint4 av = *reinterpret_cast<const uint4*>(a);
                const uint4 bv = *reinterpret_cast<const uint4*>(b);
                const uint32_t aw[4] = {av.x, av.y, av.z, av.w};
                const uint32_t bw[4] = {bv.x, bv.y, bv.z, bv.w};
                uint32_t ow[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float lo = bf16_to_f32(aw[k] & 0xffffu) * act_sigma_prime<true>(act, bf16_to_f32(bw[k] & 0xffffu));
                    const float hi = bf16_to_f32(aw[k] >> 16) * act_sigma_prime<true>(act, bf16_to_f32(bw[k] >> 16));
                    ow[k] = pack_bf16x2(lo, hi);
                }
                *reinterpret_cast<uint4*>(o) = make_uint4(ow[0], ow[1], ow[2], ow[3]);
            } else {
                for (int e = 0; e < valid; ++e)
                    o[e] = (uint16_t)f32_to_bf16(bf16_to_f32(a[e]) * act_sigma_prime<true>(act, bf16_to_f32(b[e])));
            }
        } else {
            const float* a = reinterpret_cast<const float*>(dy) + t * lddy + c0;
            const float* b = reinterpret_cast<const float*>(p) + t * ldp + c0;
            float* o = reinterpret_cast<float*>(out) + t * ldo + c0;
            if (vec && valid == V) {
                const float4 av = *reinterpret_cast<const float4*>(a);
                const float4 bv = *reinterpret_cast<const float4*>(b);
                *reinterpret_cast<float4*>(o) =
                    make_float4(av.x * act_sigma_prime<false>(act, bv.x), av.y * act_sigma_prime<false>(act, bv.y),
                                av.z * act_sigma_prime<false>(act, bv.z), av.w * act_sigma_prime<false>(act, bv.w));
            } else {
                for (int e = 0; e < valid; ++e) o[e] = a[e] * act_sigma_prime<false>(act, b[e]);
            }
        }
    }
}

unsigned grid_for(int64_t work) {
    int64_t g = (work + 255) / 256;
    if (g < 1) g = 1;
    if (g > 4096) g = 4096;
    return (unsigned)g;
}

}  // namespace

// Whether the chunk-parallel kernel takes a reduction (the same order, so
// the same bits, as the one-thread-per-group kernel).
static bool chunks_ok(const float* part, int64_t stride, const float* out, int64_t n, int splits) {
    return splits > kChunk && splits <= kChunk * kMaxChunks && n % 4 == 0 && reduce_vec_ok(part, stride, out);
}
static int64_t chunk_blocks(int64_t n) { return (n / 4 + 256 / kChunkLanes - 1) / (256 / kChunkLanes); }

hipError_t launch_reduce(const ReduceJob* jobs, int n, int splits, hipStream_t s) {
    if (n < 1 || n > kReduceBatch) return hipErrorInvalidValue;
    ReduceBatch bt;
    bt.n = n;
    bt.splits = splits;
    bool chunks = true;
    for (int i = 0; i < n; ++i) chunks = chunks && chunks_ok(jobs[i].part, jobs[i].n, jobs[i].out, jobs[i].n, splits);
    int64_t blocks = 0;
    for (int i = 0; i < n; ++i) {
        if (jobs[i].n <= 0) return hipErrorInvalidValue;
        bt.j[i] = jobs[i];
        bt.first[i] = blocks;
        blocks += chunks ? chunk_blocks(jobs[i].n) : (int64_t)grid_for((jobs[i].n + 3) / 4);
    }
    for (int i = n; i <= kReduceBatch; ++i) bt.first[i] = blocks;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if (chunks) hipLaunchKernelGGL(reduce_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, bt);
    else hipLaunchKernelGGL(reduce_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s, bt);
    return hipGetLastError();
}

hipError_t launch_pack_rows(const void* src, int64_t src_ld, int64_t rows, int64_t width, void* dst, int64_t ld,
                            hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    int shift = 3;                                           // 8 threads: a 128-byte line
    while (shift < 8 && (int64_t(1) << shift) < ld / 8) ++shift;
    int64_t grid = (rows + (256 >> shift) - 1) / (256 >> shift);
    if (grid > 8192) grid = 8192;
    hipLaunchKernelGGL(pack_rows_kernel, dim3((unsigned)grid), dim3(256), 0, s, reinterpret_cast<const uint16_t*>(src),
                       src_ld, rows, width, reinterpret_cast<uint16_t*>(dst), ld, shift);
    return hipGetLastError();
}

hipError_t launch_outer_grad(bool bf16, const void* dy, int64_t lddy, const void* p, int64_t ldp, void* out,
                             int64_t ldo, int64_t T, int64_t n, int act, hipStream_t s) {
    if (T <= 0 || n <= 0) return hipSuccess;
    const int64_t V = bf16 ? 8 : 4;
    auto al = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
    const int vec = al(dy) && al(p) && al(out) && lddy % V == 0 && ldp % V == 0 && ldo % V == 0;
    const unsigned grid = grid_for(T * ((n + V - 1) / V));
    if (bf16)
        hipLaunchKernelGGL(outer_grad_kernel<true>, dim3(grid), dim3(256), 0, s, dy, lddy, p, ldp, out, ldo, T, n,
                           act, vec);
    else
        hipLaunchKernelGGL(outer_grad_kernel<false>, dim3(grid), dim3(256), 0, s, dy, lddy, p, ldp, out, ldo, T, n,
                           act, vec);
    return hipGetLastError();
}

hipError_t launch_fill_zero(float* out, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(n)), dim3(256), 0, s, out, n);
    return hipGetLastError();
}

}  // namespace cola
