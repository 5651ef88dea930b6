// gemm_mid.hip -- the small-tile bf16 MFMA GEMM: C[M][N] = sum_k P(m, k) Q(n, k)
// with fp32 accumulation and the transposed-accumulator epilogues of
// epilogue.hpp, for outputs whose 256 x 256 tiles leave most CUs idle.
//
// Design (CDNA4, wave64, 4 waves in a 2 x 2 grid):
//  * Tiles 128 x 128, 128 x 64 and 64 x 64; each wave owns a quarter as
//    32x32x16 MFMA tiles with the Q fragment as first operand (transposed
//    accumulators, as in gemm_pp.hip), summed over k in increasing order, so
//    the values are bitwise those of the 256 x 256 family.
//  * K tiles are 64 deep (whole 128-byte lines per load row) in a ring of NS
//    LDS slots filled by direct-to-LDS loads.  The fragments of K tile kt + 1
//    are read into a second register set while the MFMAs of K tile kt run, so
//    a wave meets one barrier per K tile and its MFMAs never wait for LDS;
//    the slot of K tile kt is free at that barrier (its fragments are in
//    registers) and takes K tile kt + NS at once.
//  * What bounds a K tile: the direct-to-LDS loads touch about 0.45 128-byte
//    lines per clock per CU, so 256, 192 and 128 rows cost about 570, 430 and
//    280 clocks; the MFMAs 512, 256 and 128.  Small tiles move more bytes per
//    flop and are chosen only where they put more CUs to work.
//  * Up to kMidBatch products of one kind share a launch (the projections of
//    a group): blocks [first[i], first[i + 1]) are the tiles of product i.
//  * A partial last K tile goes through guarded registers; operands need
//    16-byte aligned rows (the dispatch falls back otherwise).
#include "internal.hpp"
#include "device_math.hpp"
#include "epilogue.hpp"
#include "lds_tile.hpp"

namespace cola {
namespace {

constexpr int BK = 64;
constexpr int NSUB = BK / 16;
constexpr int NTHR = 256;

// Operand tile of R rows (R = 64 or 128) x 64 k in LDS.
template <int R, int LAYOUT>
struct MTile;

// k-contiguous: [R rows][64 k], 128-byte rows, 16-byte chunk c of row r at
// chunk c ^ ((r >> 1) & 7)
template <int R>
struct MTile<R, KMAJ> {
    static constexpr int BYTES = R * 128;
    static constexpr int DPW = BYTES / 1024 / 4;      // 1 KB direct-to-LDS instructions per wave
    static constexpr int NL = NSUB;                   // per-lane fragment offsets: one per k step
    __device__ static __forceinline__ uint32_t voff(int blk, int64_t ld, int64_t row0, int64_t rows, int lane) {
        const int row = 8 * blk + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        const int64_t lim64 = rows - 1 - row0;
        const int lim = lim64 < R - 1 ? (int)lim64 : R - 1;
        return 2u * ((uint32_t)(row < lim ? row : lim) * (uint32_t)ld + 8u * (uint32_t)c);
    }
    __device__ static __forceinline__ const char* gbase(const uint16_t* p, int64_t ld, int64_t row0, int64_t k0) {
        return reinterpret_cast<const char*>(p + row0 * ld + k0);
    }
    __device__ static __forceinline__ void guarded(char* lds, const uint16_t* p, int64_t ld, int64_t row0,
                                                   int64_t rows, int64_t k0, int64_t kend) {
#pragma unroll
        for (int i = 0; i < R * 8 / NTHR; ++i) {
            const int id = threadIdx.x + NTHR * i;
            const int64_t row = row0 + (id >> 3), k = k0 + 8 * (id & 7);
            const int64_t valid = row < rows ? kend - k : 0;
            const uint4 v = load8_guarded(p + (row < rows ? row : 0) * ld + (valid > 0 ? k : 0),
                                          (int)(valid < 0 ? 0 : (valid > 8 ? 8 : valid)));
            const int r = id >> 3;
            *reinterpret_cast<uint4*>(lds + r * 128 + (((id & 7) ^ ((r >> 1) & 7)) << 4)) = v;
        }
    }
    // fragment of rows row0 .. row0 + 31 (row0 a multiple of 32), k step s
    __device__ static __forceinline__ uint32_t lane_off(int s, int, int lane) {
        const int r = lane & 31;
        return (uint32_t)(r * 128 + (((2 * s + (lane >> 5)) ^ ((r >> 1) & 7)) << 4));
    }
    __device__ static __forceinline__ bf16x8 frag(const char* lds, int row0, int, int s, const uint32_t (&l)[NL]) {
        return *reinterpret_cast<const bf16x8*>(lds + row0 * 128 + l[s]);
    }
};

// m-contiguous: [64 k][R m], 2R-byte rows; chunk c of row k at chunk c ^ 4 s(k)
// with s = k & 3 (R = 128: four 256-byte rows cover the banks once) or
// (k >> 1) & 1 (R = 64: two rows per 256 bytes), so that the 4 rows x 64 bytes
// a half-wave reads fall into distinct banks
template <int R>
struct MTile<R, MNMAJ> {
    static constexpr int BYTES = R * 128;
    static constexpr int DPW = BYTES / 1024 / 4;
    static constexpr int CPR = R / 8;                 // chunks per k row
    static constexpr int NL = R / 64;                 // per-lane fragment offsets: one per 32-column block
    __device__ static __forceinline__ int swz(int k) { return R == 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; }
    __device__ static __forceinline__ uint32_t voff(int blk, int64_t ld, int64_t m0, int64_t rows, int lane) {
        const int k = (64 / CPR) * blk + lane / CPR;
        const int c = (lane % CPR) ^ swz(k);
        const int64_t lim64 = (((rows - 1) >> 3) << 3) - m0;       // last chunk's first column, relative to m0
        const int lim = lim64 < R ? (int)lim64 : R;
        const int m = 8 * c <= lim ? 8 * c : lim;
        return 2u * ((uint32_t)k * (uint32_t)ld + (uint32_t)m);
    }
    __device__ static __forceinline__ const char* gbase(const uint16_t* p, int64_t ld, int64_t m0, int64_t k0) {
        return reinterpret_cast<const char*>(p + k0 * ld + m0);
    }
    __device__ static __forceinline__ void guarded(char* lds, const uint16_t* p, int64_t ld, int64_t m0, int64_t rows,
                                                   int64_t k0, int64_t kend) {
#pragma unroll
        for (int i = 0; i < BK * CPR / NTHR; ++i) {
            const int id = threadIdx.x + NTHR * i;
            const int64_t k = k0 + id / CPR, m = m0 + 8 * (id % CPR);
            const int64_t valid = k < kend ? rows - m : 0;
            const uint4 v = load8_guarded(p + (k < kend ? k : 0) * ld + (valid > 0 ? m : 0),
                                          (int)(valid < 0 ? 0 : (valid > 8 ? 8 : valid)));
            const int kr = id / CPR;
            *reinterpret_cast<uint4*>(lds + kr * (2 * R) + (((id % CPR) ^ swz(kr)) << 4)) = v;
        }
    }
    // columns 32 (b0 + j) .., k step s, by two transposing reads (see lds_tile.hpp)
    __device__ static __forceinline__ uint32_t lane_off(int j, int b0, int lane) {
        const int g = lane >> 4, i = lane & 15;
        const int kr = 8 * (g >> 1) + (i >> 2);
        const int c = 4 * (b0 + j) + 2 * (g & 1) + ((i & 3) >> 1);
        return (uint32_t)(kr * (2 * R) + ((c ^ swz(kr)) << 4) + 8 * (i & 1));
    }
    __device__ static __forceinline__ bf16x8 frag(const char* lds, int, int j, int s, const uint32_t (&l)[NL]) {
        const char* p = lds + 16 * (2 * R) * s + l[j];
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr4_t)p);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lptr4_t)(p + 4 * (2 * R)));
        const s16x8 s8 = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, s8);
    }
};

// n / d for 0 <= n < 2^22, 0 < d < 2^22, both wave-uniform: hardware
// reciprocal, then a correction of at most one either way
__device__ __forceinline__ int fdiv(int n, int d) {
    uint32_t q = (uint32_t)((float)(uint32_t)n * __builtin_amdgcn_rcpf((float)(uint32_t)d));
    const int r = n - (int)q * d;
    if (r < 0) --q;
    else if (r >= d) ++q;
    return __builtin_amdgcn_readfirstlane((int)q);
}

struct MidBatch {
    GemmArgs a[kMidBatch];
    int first[kMidBatch + 1];
    int n;
};

// LDS of a workgroup.
template <int BM, int BN, int NS>
constexpr int mid_smem_bytes() {
    return NS * (BM + BN) * 128;
}

// This block's number with an XCD-aware renumbering (block b runs on XCD b % 8):
// contiguous tiles per XCD; and the product it falls in.
__device__ __forceinline__ int mid_block(const MidBatch& bt, int* product) {
    const int nb = (int)gridDim.x;
    int b = (int)blockIdx.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    int pi = 0;
    while (pi + 1 < bt.n && b >= bt.first[pi + 1]) ++pi;
    *product = pi;
    return b - bt.first[pi];
}

// Output tile (and split) number b of the product a.
template <int BM, int BN, int NS, int PL, int QL, int EPI>
__device__ __forceinline__ void mid_tile(const GemmArgs& a, int b, char* smem) {
    using TP = MTile<BM, PL>;
    using TQ = MTile<BN, QL>;
    constexpr int TM = BM / 64, TN = BN / 64;                  // 32 x 32 tiles per wave
    constexpr int STAGE = TP::BYTES + TQ::BYTES;
    constexpr int OPS = TP::DPW + TQ::DPW;                     // loads per wave per K tile
    constexpr int NMFMA = NSUB * TM * TN;
    constexpr int NFRAG = NSUB * (TM + TN);

    const int tiles_n = (int)((a.N + BN - 1) / BN);
    const int per_split = tiles_n * (int)((a.M + BM - 1) / BM);
    const int split = a.splits > 1 ? fdiv(b, per_split) : 0;
    const int rem = b - split * per_split;
    const int tm = fdiv(rem, tiles_n);
    const int64_t m0 = (int64_t)tm * BM;
    const int64_t n0 = (int64_t)(rem - tm * tiles_n) * BN;
    const int64_t kbeg = (int64_t)split * a.k_chunk;
    const int64_t kend = min(a.K, kbeg + a.k_chunk);
    const int nk = (int)((kend - kbeg) / BK);                  // whole K tiles
    const bool tail = kbeg + (int64_t)nk * BK < kend;

    const uint16_t* P = reinterpret_cast<const uint16_t*>(a.p);
    const uint16_t* Q = reinterpret_cast<const uint16_t*>(a.q);
    const int wave = wave_id();
    const int lane = threadIdx.x & 63;
    const int wm = wave >> 1, wn = wave & 1;

    uint32_t vp[TP::DPW], vq[TQ::DPW];
#pragma unroll
    for (int j = 0; j < TP::DPW; ++j) vp[j] = TP::voff(TP::DPW * wave + j, a.ldp, m0, a.M, lane);
#pragma unroll
    for (int j = 0; j < TQ::DPW; ++j) vq[j] = TQ::voff(TQ::DPW * wave + j, a.ldq, n0, a.N, lane);
    const char* gp = TP::gbase(P, a.ldp, m0, kbeg);
    const char* gq = TQ::gbase(Q, a.ldq, n0, kbeg);
    const int64_t sp = PL == KMAJ ? 2 * BK : 2 * BK * a.ldp;   // bytes from a K tile to the next
    const int64_t sq = QL == KMAJ ? 2 * BK : 2 * BK * a.ldq;
    // Load j (of OPS) of this wave for the next K tile into the slot at s; after
    // the last one gp and gq move on to the K tile after.  Past the last whole K
    // tile the descriptors' range is 0: such loads touch no memory and leave
    // zeros, so the loop needs neither a branch nor a drain of its own.
    int left = nk;
    auto issue_one = [&](char* s, int j) __attribute__((always_inline)) {
        const int range = left > 0 ? 0x7fffffff : 0;
        if (j < TP::DPW)
            dtl16(rsrc_of(gp, range), vp[j < TP::DPW ? j : 0], s + 1024 * (TP::DPW * wave + j));
        else
            dtl16(rsrc_of(gq, range), vq[j < TP::DPW ? 0 : j - TP::DPW],
                  s + TP::BYTES + 1024 * (TQ::DPW * wave + j - TP::DPW));
        if (j == OPS - 1) {
            gp += sp;
            gq += sq;
            --left;
        }
    };
    auto issue = [&](char* s) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < OPS; ++j) issue_one(s, j);
    };

    uint32_t lp[TP::NL], lq[TQ::NL];
#pragma unroll
    for (int u = 0; u < TP::NL; ++u) lp[u] = TP::lane_off(u, wm * TM, lane);
#pragma unroll
    for (int u = 0; u < TQ::NL; ++u) lq[u] = TQ::lane_off(u, wn * TN, lane);

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    struct Frags {
        bf16x8 a[NSUB][TM], b[NSUB][TN];
    };
    // the slot's byte offset passes through an empty asm statement and a mask,
    // so that the constant parts of the fragment addresses fold into the LDS
    // instructions' offset fields
    auto at = [&](int slot) __attribute__((always_inline)) -> char* {
        uint32_t o = (uint32_t)slot * (uint32_t)STAGE;
        asm volatile("" : "+s"(o));
        return smem + (o & 0x3ffffu);
    };
    // fragment q of a K tile: for each k step, the TM of P and then the TN of Q
    auto read_one = [&](Frags& f, const char* ps, int q) __attribute__((always_inline)) {
        const int s = q / (TM + TN), i = q % (TM + TN);
        if (i < TM) f.a[s][i < TM ? i : 0] = TP::frag(ps, (wm * TM + i) * 32, i < TM ? i : 0, s, lp);
        else f.b[s][i < TM ? 0 : i - TM] = TQ::frag(ps + TP::BYTES, (wn * TN + i - TM) * 32, i < TM ? 0 : i - TM, s, lq);
    };
    auto read = [&](Frags& f, const char* ps) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NFRAG; ++q) read_one(f, ps, q);
    };
    auto mfma_one = [&](const Frags& f, int n) __attribute__((always_inline)) {
        const int s = n / (TM * TN), i = n / TN % TM, j = n % TN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[s][j], f.a[s][i], acc[i][j], 0, 0, 0);
    };
    auto compute = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NMFMA; ++n) mfma_one(f, n);
    };

    Frags f0, f1;
    int slot = 0;                                              // slot of K tile kt
    auto next = [](int s) { return s + 1 == NS ? 0 : s + 1; };
    // Loads into one slot and reads of another: the __restrict parameters say
    // that they don't overlap.  Without them the compiler waits for every load
    // in flight (vmcnt(0)) before a transposing read.
    auto issue_read = [&](char* __restrict wr, Frags& f, const char* __restrict rd) __attribute__((always_inline)) {
        issue(wr);
        read(f, rd);
    };
    // The same spread over the MFMAs of K tile `cur`: a burst of loads would
    // stall the wave on the address unit's queue while its matrix core idles
    // (128 x 128 tiles at K = 4096, 256 workgroups: 38 us with the burst).
    auto step = [&](char* __restrict wr, Frags& f, const char* __restrict rd, const Frags& cur)
                    __attribute__((always_inline)) {
        static_for<NMFMA>([&](auto nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            mfma_one(cur, n);
#pragma unroll
            for (int q = n * NFRAG / NMFMA; q < (n + 1) * NFRAG / NMFMA; ++q) read_one(f, rd, q);
#pragma unroll
            for (int j = n * OPS / NMFMA; j < (n + 1) * OPS / NMFMA; ++j) issue_one(wr, j);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // K tile kt from `cur`; the next one's fragments into `nxt`; K tile kt + NS
    // into the slot of kt.  At the barrier every wave has K tile kt in
    // registers and its loads of kt + 1 landed.
    auto body = [&](Frags& cur, Frags& nxt) __attribute__((always_inline)) {
        wait_vm<(NS - 2) * OPS>();
        barrier_lds();
        __builtin_amdgcn_sched_barrier(0);
        char* wr = smem + slot * STAGE;
        slot = next(slot);
        step(wr, nxt, at(slot), cur);
    };

    if (nk > 0) {
#pragma unroll
        for (int i = 0; i < NS - 1; ++i) issue(smem + i * STAGE);
        wait_vm<(NS - 2) * OPS>();
        barrier_lds();
        issue_read(smem + (NS - 1) * STAGE, f0, at(0));
        for (int kt = 0; kt < nk; kt += 2) {                   // two K tiles a turn: the register sets alternate
            body(f0, f1);
            if (kt + 1 < nk) body(f1, f0);
        }
        wait_vm<0>();                                          // no load may outlive the workgroup's LDS
    }
    if (tail) {
        const int64_t k0 = kbeg + (int64_t)nk * BK;
        barrier_lds();                                         // every wave is done with the slots
        TP::guarded(smem, P, a.ldp, m0, a.M, k0, kend);
        TQ::guarded(smem + TP::BYTES, Q, a.ldq, n0, a.N, k0, kend);
        barrier_lds();
        read(f0, at(0));
        compute(f0);
    }
    epilogue_block_t<EPI>(a, acc, m0 + wm * (BM / 2), n0 + wn * (BN / 2), lane, split);
}

template <int BM, int BN, int NS, int OCC, int PL, int QL, int EPI>
__global__ __launch_bounds__(NTHR, OCC) void gemm_mid_kernel(const MidBatch bt) {
    __shared__ __attribute__((aligned(1024))) char smem[mid_smem_bytes<BM, BN, NS>()];
    int pi;
    const int b = mid_block(bt, &pi);
    mid_tile<BM, BN, NS, PL, QL, EPI>(bt.a[pi], b, smem);
}

// dX = dZ A (product 0) and the weight gradients (the rest), which both follow
// from dZ, in one grid.
template <int BM, int BN, int NS, int OCC>
__global__ __launch_bounds__(NTHR, OCC) void gemm_mid_dxw_kernel(const MidBatch bt) {
    __shared__ __attribute__((aligned(1024))) char smem[mid_smem_bytes<BM, BN, NS>()];
    int pi;
    const int b = mid_block(bt, &pi);
    if (pi == 0) mid_tile<BM, BN, NS, KMAJ, MNMAJ, EPI_STORE>(bt.a[0], b, smem);
    else mid_tile<BM, BN, NS, MNMAJ, MNMAJ, EPI_STORE_F32>(bt.a[pi], b, smem);
}

// The batch and its block count (0: nothing to do).
hipError_t fill_batch(MidBatch& bt, const GemmArgs* a, int n, int bm, int bn, int64_t* blocks) {
    bt.n = n;
    *blocks = 0;
    for (int i = 0; i < n; ++i) {
        bt.a[i] = a[i];
        bt.first[i] = (int)*blocks;
        *blocks += ((a[i].M + bm - 1) / bm) * ((a[i].N + bn - 1) / bn) * (int64_t)a[i].splits;
        if (*blocks >= kMidBatch * kMidMaxBlocks) return hipErrorInvalidConfiguration;
    }
    for (int i = n; i <= kMidBatch; ++i) bt.first[i] = (int)*blocks;
    return hipSuccess;
}

template <int BM, int BN, int NS, int OCC, int PL, int QL, int EPI>
hipError_t launch_t(const GemmArgs* a, int n, hipStream_t s) {
    for (int i = 0; i < n; ++i)
        if (a[i].p_layout != PL || a[i].q_layout != QL || a[i].epi != EPI) return hipErrorInvalidValue;
    MidBatch bt;
    int64_t blocks;
    const hipError_t e = fill_batch(bt, a, n, BM, BN, &blocks);
    if (e != hipSuccess || blocks == 0) return e;
    hipLaunchKernelGGL((gemm_mid_kernel<BM, BN, NS, OCC, PL, QL, EPI>), dim3((unsigned)blocks), dim3(NTHR), 0, s, bt);
    return hipGetLastError();
}

template <int BM, int BN, int NS, int OCC>
hipError_t launch_dxw(const GemmArgs* a, int n, hipStream_t s) {
    for (int i = 0; i < n; ++i)
        if (a[i].p_layout != (i == 0 ? KMAJ : MNMAJ) || a[i].q_layout != MNMAJ ||
            a[i].epi != (i == 0 ? EPI_STORE : EPI_STORE_F32))
            return hipErrorInvalidValue;
    MidBatch bt;
    int64_t blocks;
    const hipError_t e = fill_batch(bt, a, n, BM, BN, &blocks);
    if (e != hipSuccess || blocks == 0) return e;
    hipLaunchKernelGGL((gemm_mid_dxw_kernel<BM, BN, NS, OCC>), dim3((unsigned)blocks), dim3(NTHR), 0, s, bt);
    return hipGetLastError();
}

template <int PL, int QL, int EPI>
hipError_t launch_l(const GemmArgs* a, int n, int tile, hipStream_t s) {
    switch (tile) {
        case MID_128x128: return launch_t<128, 128, 4, 1, PL, QL, EPI>(a, n, s);
        case MID_128x64: return launch_t<128, 64, 3, 2, PL, QL, EPI>(a, n, s);
        case MID_64x64: return launch_t<64, 64, 4, 2, PL, QL, EPI>(a, n, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_gemm_mid(const GemmArgs* a, int n, int tile, hipStream_t s) {
    if (n < 1 || n > kMidBatch) return hipErrorInvalidValue;
    switch (a[0].epi) {
        case EPI_Z_H: return launch_l<KMAJ, KMAJ, EPI_Z_H>(a, n, tile, s);
        case EPI_H: return launch_l<KMAJ, KMAJ, EPI_H>(a, n, tile, s);
        case EPI_GATE: return launch_l<KMAJ, KMAJ, EPI_GATE>(a, n, tile, s);
        case EPI_DGATE: return launch_l<KMAJ, MNMAJ, EPI_DGATE>(a, n, tile, s);
        case EPI_DZ: return launch_l<KMAJ, MNMAJ, EPI_DZ>(a, n, tile, s);
        case EPI_STORE_F32: return launch_l<MNMAJ, MNMAJ, EPI_STORE_F32>(a, n, tile, s);
        case EPI_STORE:
            return a[0].q_layout == KMAJ ? launch_l<KMAJ, KMAJ, EPI_STORE>(a, n, tile, s)
                                         : launch_l<KMAJ, MNMAJ, EPI_STORE>(a, n, tile, s);
        default: return hipErrorNotSupported;
    }
}

hipError_t launch_gemm_mid_dxw(const GemmArgs* a, int n, int tile, hipStream_t s) {
    if (n < 2 || n > kMidBatch) return hipErrorInvalidValue;
    switch (tile) {
        case MID_128x64: return launch_dxw<128, 64, 3, 2>(a, n, s);
        case MID_64x64: return launch_dxw<64, 64, 4, 2>(a, n, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cola
