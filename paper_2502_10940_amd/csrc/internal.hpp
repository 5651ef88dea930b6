// internal.hpp -- declarations shared by the translation units of libcola.so.
// Not part of the public ABI (that is include/cola.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cola {

// Operand layout of a GEMM C[M][N] = sum_k P(m, k) Q(n, k):
//   KMAJ : element (m, k) at ptr[m * ld + k]   (k contiguous)
//   MNMAJ: element (m, k) at ptr[k * ld + m]   (m contiguous, k strided)
enum Layout : int { KMAJ = 0, MNMAJ = 1 };

// Epilogue applied to the fp32 accumulator tile.
enum Epilogue : int {
    EPI_STORE = 0,     // c = acc, in the output dtype (bf16 / fp32 for GEMMs in fp32 storage)
    EPI_STORE_F32 = 1, // c = acc as fp32 (weight gradients, split-K partials)
    EPI_Z_H = 2,       // c = Z = round(acc); aux = H = round(sigma(Z))
    EPI_DZ = 3,        // c = dZ = round(acc * sigma'(Z)), Z read from zin; aux = H if non-NULL
    EPI_H = 4,         // c = H = round(sigma(round(acc))): H of EPI_Z_H without storing Z (inference)
    // the gated MLP of the decoder block (PP and MID kernels only):
    EPI_GATE = 5,      // c = u = round(acc) (not stored when c is NULL); aux = m = round(g u), g read from zin
    EPI_DGATE = 6,     // with dm = round(acc): c = round(dm u), aux = round(dm g); g from zin, u from zin2
};

// Which step of the layer a GEMM is (same numbering as the kernel classes of
// the public timing API).
enum Tag : int {
    TAG_FWD_Z = 0, TAG_FWD_Y = 1, TAG_BWD_DZ = 2, TAG_BWD_DX = 3, TAG_BWD_DA = 4,
    TAG_BWD_DB = 5, TAG_DENSE_FWD = 7, TAG_DENSE_DX = 8, TAG_DENSE_DW = 9, TAG_INFER_H = 11,
    TAG_FWD_YP = 12,    // K2 of the both-sigma variant: EPI_Z_H storing P and sigma_out(P)
    TAG_FWD_YG = 13,    // K2 of the up projection with the gated product (EPI_GATE)
    TAG_BWD_DXG = 14    // K4 of the down projection with the gated product's backward (EPI_DGATE)
};

struct GemmArgs {
    int64_t M, N, K;
    const void* p; int64_t ldp; int p_layout;    // left operand P
    const void* q; int64_t ldq; int q_layout;    // right operand Q (C = P Q^T)
    void* c; int64_t ldc;                        // output
    void* aux; int64_t ldaux;                    // second output (H) or NULL
    const void* zin; int64_t ldzin;              // Z read by EPI_DZ, g by EPI_GATE / EPI_DGATE
    const void* zin2; int64_t ldzin2;            // u read by EPI_DGATE
    int epi;
    int tag;                                     // Tag
    int act;                                     // 0 identity, 1 SiLU
    int splits;                                  // split-K count (>= 1)
    int64_t k_chunk;                             // K range per split (multiple of the K tile)
    int64_t split_stride;                        // elements between partial slices of c
    int route;                                   // Route: ROUTE_AUTO, or the one a weight-gradient split was planned for
};

// Enqueue one GEMM.  Return hipSuccess or the launch error.
hipError_t launch_gemm_bf16(const GemmArgs& a, hipStream_t s);
// n products of one kind (same tag, all unsplit), in shared launches where that is
// faster.
hipError_t launch_gemm_bf16_batch(const GemmArgs* a, int n, hipStream_t s);
// The kernel families behind launch_gemm_bf16:
//   STREAM -- BM x 128 tiles, direct-to-LDS loads, three K stages, two per CU
//   PP     -- 256 x 256 tiles, two wave groups per workgroup in ping-pong
hipError_t launch_gemm_stream(const GemmArgs& a, hipStream_t s);
hipError_t launch_gemm_pp(const GemmArgs& a, hipStream_t s);
// n products of one kind (n <= kMidBatch; both operands m-contiguous and fp32
// output, or EPI_STORE of k-contiguous operands, or EPI_DZ) in one PP grid, one
// workgroup per tile and split.
hipError_t launch_gemm_pp_batch(const GemmArgs* a, int n, hipStream_t s);
// n weight-gradient products planned for one route (n <= kMidBatch): one launch
// when their operands are aligned (else one each, as launch_gemm_bf16).
hipError_t launch_gemm_bf16_wgrads(const GemmArgs* a, int n, hipStream_t s);
// dX = dZ A (a[0]) and the weight gradients a[1 ..] in one launch: whether that is
// the faster way, and the launch.
bool bf16_dxw_takes(const GemmArgs* a, int n);
hipError_t launch_gemm_bf16_dxw(const GemmArgs* a, int n, hipStream_t s);

//   MID -- 128 x 128, 128 x 64 or 64 x 64 tiles, for outputs too small for PP;
//   n products of one kind (same layouts and epilogue; n <= kMidBatch) in one
//   launch, each of fewer than kMidMaxBlocks tiles.
enum MidTile : int { MID_128x128 = 0, MID_128x64 = 1, MID_64x64 = 2 };
constexpr int kMidBatch = 4;
constexpr int64_t kMidMaxBlocks = int64_t(1) << 20;
hipError_t launch_gemm_mid(const GemmArgs* a, int n, int tile, hipStream_t s);
// dX = dZ A (a[0]) and the weight gradients a[1 ..] of a small layer in one grid
// (MID_128x64 or MID_64x64).
hipError_t launch_gemm_mid_dxw(const GemmArgs* a, int n, int tile, hipStream_t s);
//   SKINNY -- at most kSkinnyRows token rows against weight rows (both
//   k-contiguous, any alignment); n products of one kind and the same tokens in
//   one launch (n <= kMidBatch).
constexpr int64_t kSkinnyRows = 32;
hipError_t launch_gemm_skinny(const GemmArgs* a, int n, hipStream_t s);
// Whether the forward products of M tokens run there.
bool skinny_rows(int64_t M);

// Kernel and tile of a bf16 product.
enum Route : int {
    ROUTE_AUTO = 0,        // GemmArgs: let the launcher choose
    ROUTE_STREAM, ROUTE_PP, ROUTE_MID_128x128, ROUTE_MID_128x64, ROUTE_MID_64x64,
    ROUTE_SKINNY           // forward products of at most kSkinnyRows tokens
};
// Route of an unsplit product with aligned operands: the fastest by the cost
// model of gemm_dispatch.hip; the option OPT_STREAM_ONLY sends every product
// to STREAM.
int gemm_route(int64_t M, int64_t N, int64_t K);
// The route that the option OPT_TILE asks for, where it fits; ROUTE_AUTO: none.
int asked_route();
// Modelled microseconds of `tiles` output tiles (splits included) of `steps`
// 64-deep K tiles each on a PP or MID route; wgrad: both operands m-contiguous.
double route_us(int route, int64_t tiles, int64_t steps, bool wgrad);
// Whether a PP or MID route takes an M x N product in `splits` splits: PP at
// least 128 x 128 (half a tile), MID fewer than kMidMaxBlocks tiles (its block
// arithmetic).
bool route_fits(int route, int64_t M, int64_t N, int64_t splits);
// Output tiles of an M x N product on a PP or MID route.
int64_t route_tiles(int route, int64_t M, int64_t N);
// Whether a PP or MID kernel (not STREAM) runs this GEMM: the gated epilogues
// exist only there.
bool fused_epilogue_takes(const GemmArgs& a);

// Process-wide tuning options (the public cola_set_option): the values of
// cola_option in include/cola.h.  set_option returns 0, or -1 for an unknown
// option or value.
enum Option : int { OPT_STREAM_ONLY = 0, OPT_WGRAD_PAIR = 1, OPT_FUSE_GATE = 2, OPT_TILE = 3 };
int set_option(int option, int value);
int get_option(int option);

// fp32 storage: n products of one kind (same layouts and epilogue) in one launch.
constexpr int kF32Batch = 4;
hipError_t launch_gemm_f32_batch(const GemmArgs* a, int n, hipStream_t s);
// dX = dZ A (a[0]) and the weight gradients a[1 ..] of a small layer in one grid of
// 32 x 32 tiles, and whether both parts would use that tile anyway.
bool f32_dxw_takes(const GemmArgs* a, int n);
hipError_t launch_gemm_f32_dxw(const GemmArgs* a, int n, hipStream_t s);
// tb x tb output tiles of an M x N product.
inline int64_t f32_tiles(int64_t tb, int64_t M, int64_t N) { return ((M + tb - 1) / tb) * ((N + tb - 1) / tb); }

// out[i] = sum_{k < splits} part[k * n + i], i < n, in a fixed order of k (fp32);
// up to kReduceBatch of them with one split count in a launch.
constexpr int kReduceBatch = 4;
struct ReduceJob {
    const float* part;
    float* out;
    int64_t n;
};
hipError_t launch_reduce(const ReduceJob* jobs, int n, int splits, hipStream_t s);
// dst[r][c] = src[r][c] for c < width, 0 for width <= c < ld (16-bit elements;
// src rows src_ld apart, any alignment; dst 16-byte aligned, ld a multiple of
// 8).  Gives operands with odd widths or pitches aligned rows.
hipError_t launch_pack_rows(const void* src, int64_t src_ld, int64_t rows, int64_t width, void* dst, int64_t ld,
                            hipStream_t s);
// out[i] = 0 for i < n (fp32 words).
hipError_t launch_fill_zero(float* out, int64_t n, hipStream_t s);

// out[t][o] = dy[t][o] * sigma_act'(p[t][o]) over T rows of n elements, in
// the storage dtype (bf16 rounded to nearest even, or fp32).
hipError_t launch_outer_grad(bool bf16, const void* dy, int64_t lddy, const void* p, int64_t ldp, void* out,
                             int64_t ldo, int64_t T, int64_t n, int act, hipStream_t s);

// Largest row pitch (elements) of any operand: the 256 x 256 family reads a
// K tile of a k-contiguous operand through a buffer descriptor whose range is
// 2^31 bytes from the tile's first row, and 255 rows of this pitch fit it.
// Descriptors with wider pitches are refused (COLA_ERR_BAD_SHAPE).
constexpr int64_t kMaxPitch = int64_t(1) << 22;

// K tile of the bf16 kernel: split-K chunks are multiples of it.
constexpr int BF16_BK = 64;
// K tile of the fp32 kernel.
constexpr int F32_BK = 32;

}  // namespace cola
