// Host-side launchers of the gfx950 kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace espace {

enum TileKind {
    TILE_128x128 = 3,        // gemm_bf16_v2.hip, 4 waves as 2 x 2
    TILE_256x256 = 5,        // gemm_bf16_v3.hip, 4 waves as 2 x 2 (128 x 128 each)
    TILE_128x192 = 6,        // gemm_bf16_v2.hip, 8 waves as 4 x 2; long depths as below
    TILE_256x192 = 7,        // gemm_bf16_v3.hip, 4 waves as 2 x 2 (128 x 96 each)
    TILE_192x192 = 8,        // gemm_bf16_v4.hip, 8 waves as 2 x 2 x 2 depth halves
    TILE_256x160 = 9,        // the same
};

// Limit of the bounded cross-workgroup waits and the device counter of the
// waits that gave up (see note_timeout).
struct WaitCfg {
    unsigned spins = 1u << 22;
    unsigned long long* timeouts = nullptr;
};

// One "TN" product C[r][c] = sum_k A[r][k] * B[c][k]  (bf16 in, fp32 accumulate).
struct GemmArgs {
    const uint16_t* A;
    int64_t lda;
    const uint16_t* B;
    int64_t ldb;
    void* C;            // bf16 output (or fp32 when c_f32)
    int64_t ldc;
    int R;              // rows of A and C
    int Cc;             // rows of B = columns of C
    int D;              // reduced dimension
    int c_f32;          // 1: write fp32 output
    int tile;           // TileKind
    int splits;         // depth ranges; > 1 needs `partial`
    float* partial;     // splits * R * splitk_ld(Cc) fp32 (workspace); with `pair`:
                        // tiles * tile area fp32, then one 8-byte state word per tile
    int cus = 256;      // compute units of the device (persistent grids)
    WaitCfg wait;       // bounded waits of the pair combine
    int pair = 0;       // splits == 2 combined inside the kernel (no reduce pass)
    unsigned long long epoch = 0;   // per-call tag of the pair state words
    // Row-pair layout (a matrix the library keeps to itself: Z in the layer's
    // workspace).  Element (r, k) sits at (r / 2) * ld + (k / 32) * 64 +
    // (r % 2) * 32 + k % 32: every 128-byte block holds 32 consecutive
    // elements of two neighbouring rows, so a 32-deep load of a row pair is
    // one whole cache line.  ld (elements per row pair) is a multiple of 64.
    int a_pairs = 0;    // A is in the row-pair layout (lda its pair pitch)
    int c_pairs = 0;    // write C (bf16) in the row-pair layout (ldc its pair pitch)
};

// Whether all XCDs walk the depth of a tiled product in one order (DepthOrder of
// common.hpp gives each its own start).  256 x 256 and 128 x 128 tiles from 320 MB of
// operands or 16384 of depth on: past the 256 MB Infinity Cache a panel that several
// XCDs read is found there only if they read it at about the same time.  Over 44 such
// sizes an order per XCD cost 256 x 256 tiles 1.3% (1180 x 22272 x 20168: 1394 -> 1528
// us, 6144 x 2458 x 24576: 597 -> 610), 128 x 128 ones 2.8%; over the 124 others it saved
// 2.3 and 2.0%.
inline bool one_depth_order(const GemmArgs& g, int bm, int bn) {
    return bm == bn && (((int64_t)g.R + g.Cc) * g.D >= 160000000 || g.D >= 16384);
}

// Bits of the tiled kernels' `map` argument next to those of tile_coords
constexpr int MAP_ONE_ORDER = 16;                 // one depth order for all XCDs

// offset (elements) of element (r, k) of a row-pair matrix with pair pitch ld
__host__ __device__ inline int64_t pair_offset(int64_t r, int64_t k, int64_t ld) {
    return (r >> 1) * ld + (k >> 5) * 64 + (r & 1) * 32 + (k & 31);
}

// Tiles of bm x bn of an n x n matrix that reach the diagonal or lie above it:
// the first such tile column of tile row r, and their number.
__host__ __device__ inline int upper_first(int r, int bm, int bn) { return r * bm / bn; }
inline int upper_tiles(int n, int bm, int bn) {
    const int tr = (n + bm - 1) / bm, tc = (n + bn - 1) / bn;
    int t = 0;
    for (int r = 0; r < tr; ++r) t += tc - upper_first(r, bm, bn);
    return t;
}

// Tile size of a TileKind in the pair-combine kernel (rows, columns).
void tile_dims(int tile, int* bm, int* bn);

// leading dimension of split-K partial sums
inline int64_t splitk_ld(int Cc) { return (Cc + 7) / 8 * 8; }

hipError_t launch_gemm_tn_bf16(const GemmArgs& g, hipStream_t stream);
hipError_t launch_gemm_tn_bf16_v2(const GemmArgs& g, hipStream_t stream);
// Eight waves that halve every step: 192 x 192 and 256 x 160 tiles, and 128 x 192
// ones at V4_MIN_STEPS steps of 64 or more per range.  hipErrorInvalidValue for
// 2^31 elements or more.
constexpr int V4_MIN_STEPS = 48;
hipError_t launch_gemm_tn_bf16_v4(const GemmArgs& g, hipStream_t stream);
// Four-wave 256 x 256 and 256 x 192 kernel with a hand-ordered main loop;
// hipErrorInvalidValue for products it does not take (other tiles, fp32
// output, >= 2^31 elements).
hipError_t launch_gemm_tn_bf16_v3(const GemmArgs& g, hipStream_t stream);
// Small-tile product for a few to a few hundred tokens (tile: index of the
// configuration mid_plan chose; splits > 1 needs `partial`).  mid_plan, for up to
// `ranges` depth ranges, returns the estimated time in us; mid_supported says
// whether the leading dimensions fit its 32-bit offsets, mid_waves into how many
// sums a configuration's waves split a range.
double mid_plan(int R, int Cc, int D, int cus, int ranges, int* config, int* splits);
int mid_waves(int config);
bool mid_supported(int64_t lda, int64_t ldb);
hipError_t launch_mid_tn_bf16(const GemmArgs& g, hipStream_t stream);
// Vector-ALU product for 1 <= R <= 2 tokens with whole-row streaming (tile,
// splits, partial unused); gemv_supported says whether the tokens fit its LDS.
bool gemv_supported(int R, int D);
hipError_t launch_gemv_tn_bf16(const GemmArgs& g, hipStream_t stream);
// Persistent streaming product for up to 16 tokens with the many-row operand
// streamed through an LDS ring (tile, splits, partial unused); stream_supported
// says whether the tokens and depth fit (depth up to 6144).
bool stream_supported(int R, int D);
hipError_t launch_stream_tn_bf16(const GemmArgs& g, hipStream_t stream);
// Upper triangle of a symmetric product (A = B): fp32 sums of g.splits depth ranges
// at g.partial + s * R * splitk_ld(Cc), not combined; the 32 x 32 blocks wholly
// below the diagonal may not be computed.
hipError_t launch_mid_tn_bf16_ranges(const GemmArgs& g, hipStream_t stream);
// out_bf16: 0 fp32 output, 1 bf16, 2 bf16 in the row-pair layout
hipError_t launch_splitk_reduce(const float* P, int S, int64_t split_stride, int64_t ldp,
                                void* C, int64_t ldc, int R, int Cc, int out_bf16,
                                hipStream_t stream);
hipError_t launch_gemm_tn_f32(const float* A, int64_t lda, const float* B, int64_t ldb,
                              float* C, int64_t ldc, int R, int Cc, int D, int cus, hipStream_t stream);

// fp32 sums of the depth ranges of a 256 x 256 or 256 x 192 tiled product
// (g.splits ranges requested; *ranges receives the number of non-empty ones),
// range s at g.partial + s * R * splitk_ld(Cc); not combined.  upper (R == Cc):
// just the tiles that reach the diagonal or lie above it.
hipError_t launch_gemm_tn_bf16_v3_ranges(const GemmArgs& g, bool upper, int* ranges, hipStream_t stream);

// Calibration (autocorrelation of calibration tokens, principal components).
int autocorr_ranges(int64_t M, int64_t K, bool f32, int cus);
size_t autocorr_workspace_bytes(int64_t M, int64_t K, bool f32, int cus);
hipError_t launch_autocorr_update(const void* X, int64_t ldx, int M, int K, bool f32, bool normalize,
                                  float alpha, float* C, int64_t ldc, void* workspace, int cus, hipStream_t stream);
size_t pca_workspace_bytes(int64_t K);
bool pca_available();
hipError_t launch_principal_components(const float* C, int64_t ldc, int K, int L, bool by_magnitude, void* Pt,
                                       int64_t ldp, bool f32, float* evals, int* info, void* workspace,
                                       hipStream_t stream);
size_t symprod_workspace_bytes(int64_t K);
// dst[c][r] = src[r][c] for r < rows, c < cols (bf16 or fp32; values copied
// exactly).  Both leading dimensions are multiples of 8 elements; the bf16
// kernel may write the padding columns of dst's rows (scratch only).
hipError_t launch_transpose(const void* src, int64_t lds, int rows, int cols, void* dst, int64_t ldd, bool f32,
                            hipStream_t stream);
hipError_t launch_symmetrized_product(const float* A, int64_t lda, const float* B, int64_t ldb, float* C,
                                      int64_t ldc, int K, float alpha, float beta, void* workspace, int cus,
                                      hipStream_t stream);

// ---- MX-FP8 products (gemm_mxfp8.hip) ----------------------------------------
// out[r][c] = sum_d T[r][d]·W[c][d] over MX-FP8 operands (codes with zero
// padding up to round_up(D, 128), one E8M0 scale byte per 32 along d).
struct MxGemmArgs {
    const uint8_t* T;  int64_t ldt;     // token-side codes [R][ldt]
    const uint8_t* Ts; int64_t ldts;    // its scale bytes [R][ldts]
    const uint8_t* W;  int64_t ldw;     // weight-side codes [C][ldw]
    const uint8_t* Ws; int64_t ldws;    // its scale bytes [C][ldws]
    void* out;         int64_t ldo;     // bf16 Y [R][ldo], or MX-FP8 codes [R][ldo]
    uint8_t* outs;     int64_t ldos;    // MX-FP8 output: scale bytes [R][ldos]
    int R, C, D;
    int cpad;                           // MX-FP8 output: columns written, round_up(C, 128)
    // Row pairs (the MX-FP8 layer's Z in its workspace): code (r, c) at
    // (r / 2) * ld + (c / 64) * 128 + (r % 2) * 64 + c % 64, ld (bytes per
    // row pair) a multiple of 128; the scale bytes stay one row per token.
    int t_pairs = 0;                    // the token codes T (bf16 output only)
    int out_pairs = 0;                  // the MX-FP8 output codes
};
// The projection's tile for R x C outputs at depth D, and its estimated time.
enum MxProjTile { MX_TILE_256x256, MX_TILE_128x128, MX_TILE_128x192 };
MxProjTile mx_proj_tile(int R, int C, int D, int cus, double* us);
// out_mx: write MX-FP8 (codes and scales along the columns) instead of bf16.
// hipErrorInvalidValue when an operand spans 2^31 bytes or more.
hipError_t launch_gemm_mx(const MxGemmArgs& a, int out_mx, int cus, hipStream_t stream);
// The small-tile configuration launch_gemm_mx takes for these sizes (token
// codes in plain rows), or -1: a tiled kernel.
int mx_small_config(int R, int C, int D, int cus, int out_mx);
// mid_mxfp8.hip: the cheapest small-tile configuration, -1 if none is
// estimated below tiled_us; its launch.
int mx_mid_config(int R, int C, int D, int cus, int out_mx, double tiled_us);
hipError_t launch_mx_mid(const MxGemmArgs& a, int out_mx, int config, bool scales16, hipStream_t stream);
// proj_mxfp8.hip: MX-FP8 output on 128 x 192 tiles whose waves halve every step.
hipError_t launch_proj_mx(const MxGemmArgs& a, bool scales16, hipStream_t stream);
hipError_t launch_mx_quantize(const uint16_t* A, int64_t lda, int R, int C, uint8_t* Q, int64_t ldq, uint8_t* S,
                              int64_t lds, hipStream_t stream);

}  // namespace espace
