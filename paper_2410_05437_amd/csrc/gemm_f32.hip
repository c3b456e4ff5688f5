// float32 "TN" product C[r][c] = sum_k A[r][k] * B[c][k] on the fp32 MFMA
// (the float32 layers and gradients, the calibration products).
//
// fp32 MFMA issue 256 flops per clock and CU, twice the vector ALU's rate
// without packed instructions.  In both kernels the MFMA takes the B rows as
// its first operand, so a lane ends with runs of 4 consecutive output columns
// of one row, and the depth index of an operand is permuted the same way for
// both: a lane's 16-byte chunk holds 4 consecutive k, chunk q of a row goes
// to lane group q, and MFMA e of a slab takes element e of every chunk.  The
// sums of 32 (tiled) or 8 to 16 terms are formed apart and then added, so that
// a long sum rounds at its full size that many times less often.
#include "common.hpp"
#include "kernels.hpp"

namespace espace {

namespace {

__device__ __forceinline__ f32x4_t load4_masked(const float* row, int k, int depth) {
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    const int nvalid = depth - k;
    if (nvalid >= 4) {
        v = *reinterpret_cast<const f32x4_t*>(row + k);
    } else if (nvalid > 0) {
        const f32x4_t t = *reinterpret_cast<const f32x4_t*>(row + k);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = e < nvalid ? t[e] : 0.f;
    }
    return v;
}

template <int MI> struct AccF;
template <> struct AccF<32> { typedef f32x16_t type; };
template <> struct AccF<16> { typedef f32x4_t type; };

__device__ __forceinline__ f32x16_t mfma_f32(float b, float a, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(b, a, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4_t mfma_f32(float b, float a, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(b, a, c, 0, 0, 0);
}

// Four consecutive columns c .. c + 3 of output row `row`.
__device__ __forceinline__ void store4(float* row, int c, int Cc, f32x4_t v) {
    if (c + 4 <= Cc) {
        *reinterpret_cast<f32x4_t*>(row + c) = v;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c + e < Cc) row[c + e] = v[e];
    }
}

// Tiles of BM x BN outputs, four waves as 2 x 2, each a grid of 32 x 32 blocks
// of v_mfma_f32_32x32x2_f32.  Bound by the matrix cores: a 32-deep step of a
// 128 x 128 tile is 4096 cycles of MFMA per SIMD against 32 KB of operands, so
// two LDS stages of 128-byte rows, two workgroups per CU and one barrier per
// step suffice: 4096^3 in 1030 us, 133 TFLOP/s of the 157 the matrix cores
// issue (the vector-ALU kernel before it, 64 x 64 tiles: 1760 us; 1100 x 2048
// x 2048: 172 -> 103 us; 1024^3: 65 -> 24 us).  Chunk c of row r sits at chunk c ^ ((r >> 1) & 7): the 16 rows
// that 16 neighbouring lanes read fall on all 64 banks.
constexpr int TK = 32;                            // depth step: 128-byte rows

template <int BM, int BN>
__global__ __launch_bounds__(256, 2)
void gemm_tn_f32_mfma_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
                             float* __restrict__ C, int64_t ldc, int R, int Cc, int D, int tiles_c) {
    constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 32, TN = WN / 32;
    constexpr int STAGE = (BM + BN) * TK * 4;
    constexpr int LPW = (BM + BN) / 8 / 4;        // 1 KB loads (8 rows) per wave and stage
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * STAGE];
    int tile_r, tile_c;
    tile_coords<4>(blockIdx.x, gridDim.x, tiles_c, 0, tile_r, tile_c);
    const int row0 = tile_r * BM, col0 = tile_c * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr0 = (wave >> 1) * WM, wc0 = (wave & 1) * WN;

    // descriptors over the tile's own rows (the launcher checks that these
    // span less than 2^32 bytes); rows past the matrix repeat its last row
    const int nr = min(BM, R - row0), nc = min(BN, Cc - col0);
    const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (int64_t)row0 * lda), (short)0,
                                                      (int)(uint32_t)((uint64_t)nr * lda * 4u), 0x00020000);
    const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(B + (int64_t)col0 * ldb), (short)0,
                                                      (int)(uint32_t)((uint64_t)nc * ldb * 4u), 0x00020000);
    unsigned off[LPW];
    int kc[LPW];
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
        const int q = wave + 4 * j;
        const int rl = 8 * q + (lane >> 3);
        const bool isA = 8 * q < BM;
        const int rr = isA ? rl : rl - BM;
        kc[j] = ((lane & 7) ^ ((rr >> 1) & 7)) * 4;
        const int g = isA ? min(rr, nr - 1) : min(rr, nc - 1);
        off[j] = (unsigned)(((uint64_t)g * (isA ? lda : ldb) + kc[j]) * 4u);
    }
    auto issue = [&](int t) {
        unsigned char* stage = smem + (t & 1) * STAGE;
        const int k0 = t * TK;
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
            const int q = wave + 4 * j;
            // chunks at or past the depth are read past the descriptor: zeros
            const unsigned o = k0 + kc[j] < D ? off[j] + (unsigned)k0 * 4u : 0xFFFFFFF0u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(8 * q < BM ? ra : rb,
                                                     (__attribute__((address_space(3))) void*)(stage + q * 1024), 16,
                                                     (int)o, 0, 0, 0);
        }
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int lr = lane & 31, lh = lane >> 5, sw = (lr >> 1) & 7;
    const int steps = (D + TK - 1) / TK;
    issue(0);
    for (int t = 0; t < steps; ++t) {
        // this wave's loads of step t have landed, and after the barrier
        // every wave's; every wave is done reading the other stage
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (t + 1 < steps) issue(t + 1);
        const unsigned char* stage = smem + (t & 1) * STAGE;
        const unsigned char* pa = stage + (wr0 + lr) * (TK * 4);
        const unsigned char* pb = stage + (BM + wc0 + lr) * (TK * 4);
        const int left = D - t * TK;              // only the last step has fewer than TK
        f32x16_t part[TM][TN];
#pragma unroll
        for (int s = 0; s < TK / 8; ++s) {
            const int c = ((2 * s + lh) ^ sw) * 16;
            f32x4_t fa[TM], fb[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[i] = *reinterpret_cast<const f32x4_t*>(pa + i * 32 * TK * 4 + c);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[j] = *reinterpret_cast<const f32x4_t*>(pb + j * 32 * TK * 4 + c);
            if (left < TK) {
                // the chunk that straddles the depth: its padding is not used
                const int nv = left - 8 * s - 4 * lh;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[i][e] = e < nv ? fa[i][e] : 0.f;
#pragma unroll
                    for (int j = 0; j < TN; ++j) fb[j][e] = e < nv ? fb[j][e] : 0.f;
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        part[i][j] = mfma_f32(fb[j][e], fa[i][e], s == 0 && e == 0 ? f32x16_t{} : part[i][j]);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] += part[i][j];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = row0 + wr0 + 32 * i + lr;
        if (r >= R) continue;
        float* row = C + (int64_t)r * ldc;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                store4(row, col0 + wc0 + 32 * j + 8 * q + 4 * lh, Cc,
                       f32x4_t{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]});
    }
}

// Products too small to fill the chip with tiles: one MI x MI block of the
// output per workgroup, its W waves taking turns at the depth (UD consecutive
// slabs of 256 / MI each, loaded straight to registers), the partial sums
// added in wave order through LDS.  Bound by latency, or by the stream of the
// many-row operand for a few tokens: with the depth one serial chain per tile
// the 128 x 64 x 256 projection took 17 us and 16 x 4096 x 2048 130 us, now
// below 10 us with the launch.
template <int MI, int W, int UD>
__global__ __launch_bounds__(W * 64)
void gemm_tn_f32_split_kernel(const float* __restrict__ A, int64_t lda, const float* __restrict__ B, int64_t ldb,
                              float* __restrict__ C, int64_t ldc, int R, int Cc, int D, int tiles_c) {
    using Acc = typename AccF<MI>::type;
    constexpr int SD = 256 / MI;                  // depth of a slab: one 16-byte chunk per lane
    constexpr int NQ = MI * MI / 256;             // 4-column runs per lane
    __shared__ f32x4_t red[W][NQ][64];
    int tile_r, tile_c;
    tile_coords<4>(blockIdx.x, gridDim.x, tiles_c, 0, tile_r, tile_c);
    const int row0 = tile_r * MI, col0 = tile_c * MI;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane % MI, lk = lane / MI * 4;
    const float* arow = A + (int64_t)min(row0 + lr, R - 1) * lda;
    const float* brow = B + (int64_t)min(col0 + lr, Cc - 1) * ldb;
    Acc acc;
#pragma unroll
    for (int e = 0; e < 4 * NQ; ++e) acc[e] = 0.f;
    for (int k0 = wave * UD * SD; k0 < D; k0 += W * UD * SD) {
        f32x4_t fa[UD], fb[UD];
        if (k0 + UD * SD <= D) {
#pragma unroll
            for (int u = 0; u < UD; ++u) {
                fb[u] = *reinterpret_cast<const f32x4_t*>(brow + k0 + u * SD + lk);
                fa[u] = *reinterpret_cast<const f32x4_t*>(arow + k0 + u * SD + lk);
            }
        } else {
#pragma unroll
            for (int u = 0; u < UD; ++u) {
                fb[u] = load4_masked(brow, k0 + u * SD + lk, D);
                fa[u] = load4_masked(arow, k0 + u * SD + lk, D);
            }
        }
#pragma unroll
        for (int u = 0; u < UD; ++u) {
            Acc part = {};
#pragma unroll
            for (int e = 0; e < 4; ++e) part = mfma_f32(fb[u][e], fa[u][e], part);
            acc += part;
        }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) red[wave][q][lane] = f32x4_t{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    __syncthreads();
    if (wave >= NQ) return;
    f32x4_t v = red[0][wave][lane];
#pragma unroll
    for (int w = 1; w < W; ++w) v += red[w][wave][lane];
    const int r = row0 + lr;
    if (r < R) store4(C + (int64_t)r * ldc, col0 + 8 * wave + lk, Cc, v);
}

}  // namespace


hipError_t launch_gemm_tn_f32(const float* A, int64_t lda, const float* B, int64_t ldb,
                              float* C, int64_t ldc, int R, int Cc, int D, int cus, hipStream_t stream) {
    auto tiles = [&](int t) { return (int64_t)((R + t - 1) / t) * ((Cc + t - 1) / t); };
    // the tiled kernels' 32-bit offsets inside a tile
    const bool fits = (lda > ldb ? lda : ldb) * 128 * 4 < ((int64_t)1 << 32);
    const int few = R < Cc ? R : Cc;
    auto tiled = [&](auto kernel, int t) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles(t)), dim3(256), 0, stream, A, lda, B, ldb, C, ldc, R, Cc, D,
                           (Cc + t - 1) / t);
        return hipGetLastError();
    };
    // one launch unless its 512-thread workgroups were 2^32 threads, a launch's limit
    auto split = [&](auto kernel, int t) {
        const int64_t most = 1 << 22;
        const int64_t tc = (Cc + t - 1) / t < most ? (Cc + t - 1) / t : most;
        const int64_t cols = tc * t, rows = most / tc * t;
        for (int64_t r = 0; r < R; r += rows)
            for (int64_t c = 0; c < Cc; c += cols) {
                const int nr = (int)(R - r < rows ? R - r : rows), nc = (int)(Cc - c < cols ? Cc - c : cols);
                hipLaunchKernelGGL(kernel, dim3((unsigned)(((nr + t - 1) / t) * ((nc + t - 1) / t))), dim3(512), 0,
                                   stream, A + r * lda, lda, B + c * ldb, ldb, C + r * ldc + c, ldc, nr, nc, D,
                                   (nc + t - 1) / t);
                const hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
            }
        return hipSuccess;
    };
    // Few rows or columns first: a tile's unused half or more costs as much as the
    // used one.  Up to 16 of them, 16 x 16 blocks whose waves split the depth (1 x 32768
    // x 1024 28 us, 64 x 64 tiles 41, 128 x 128 ones 74; 100000 x 8 x 512 45, 66 and 140); up
    // to 32, 32 x 32 ones (17 x 65536 x 1024 68, 75 and 135), but at shallow depths 64 x
    // 64 tiles once they are enough (24 x 65536 x 256 22 against 26, 30000 x 32 x 64 5.8
    // against 7.0; 32 x 16384 x 256 9.2 against 8.4).
    if (few <= 16) return split(gemm_tn_f32_split_kernel<16, 8, 4>, 16);
    const bool shallow = D <= 256 && tiles(64) * 128 >= (int64_t)cus * D;
    if (few <= 32 && tiles(32) >= 5 * (int64_t)cus / 8 && !(fits && shallow))
        return split(gemm_tn_f32_split_kernel<32, 8, 4>, 32);
    // 128 x 128 tiles once there is one for every CU (4096^3, 1024 tiles:
    // 1030 against 1079 us with 64 x 64 tiles; 2048 x 2048 x 8192, 256: 542
    // against 549; 1100 x 2048 x 2048, 153: 132 against 103); 64 x 64 tiles
    // from half as many as CUs (1000 x 600 x 1500, 160 tiles: 33 against 36
    // us with 32 x 32 blocks; 200 x 1024 x 1024, 64: 23 against 11).  Below
    // that the depth is split over a workgroup's waves: 32 x 32 blocks from
    // 5/8 as many as CUs (200 x 1024 x 1024, 224 blocks: 11 against 17 us
    // with 16 x 16 ones; 200 x 300 x 2000, 70: 16 against 9.5), 16 x 16
    // blocks below.
    if (fits && few > 64 && tiles(128) >= cus) return tiled(gemm_tn_f32_mfma_kernel<128, 128>, 128);
    if (fits && tiles(64) >= cus / 2) return tiled(gemm_tn_f32_mfma_kernel<64, 64>, 64);
    if (tiles(32) >= 5 * (int64_t)cus / 8) return split(gemm_tn_f32_split_kernel<32, 8, 4>, 32);
    return split(gemm_tn_f32_split_kernel<16, 8, 4>, 16);
}

}  // namespace espace
