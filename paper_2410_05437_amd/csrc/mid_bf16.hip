// bfloat16 "TN" product C[r][c] = sum_k A[r][k] * B[c][k] (fp32 accumulation)
// for a few to a few hundred tokens: decode beyond one or two tokens, batched
// decode and short prompts.
//
// These products are bound by moving operands: the many-row operand B comes
// from HBM once, and every workgroup reads the BM token rows and BN rows of B
// of its output tile through its CU's load path.  So:
//  * Small tiles (8 to 112 tokens x 8 to 96 rows of B, one of the list below)
//    give every CU work in one round without a depth split over workgroups;
//    mid_plan prices each and takes the cheapest.
//  * The W waves of a workgroup split the depth instead of the tile (wave w
//    takes the 64-deep steps w, w + W, ...), each with the whole tile in its
//    accumulators and a ring of ST LDS stages of its own, filled by
//    buffer_load ... lds and read by nobody else.  The main loop has no
//    barrier: waves drift apart, so loads and arithmetic of different waves
//    overlap by themselves and 100 to 160 KB per CU stay in flight.  The
//    partial sums are added through LDS at the end, in wave order.
//  * A stage's rows are 128 bytes, whole cache lines; the waves' steps are
//    neighbours, so together they read 512 bytes to 1 KB of a row.
// Rates: 65 to 80 KB/us per CU through the load path, or 4.5 to 5.5 TB/s of B
// from HBM; short products (8 x 1536 x 4096: data return busy 19% of the time) are
// launch, ramp and the final sums.  Each XCD starts at another depth (DepthOrder: 333 x 1536 x 11008
// 33.0 -> 31.0 us, 48 x 12288 x 4096 22.5 -> 20.7).  Measured as calls of a captured
// graph, operands rotated through HBM, the gap between two calls included, against
// the kernels used before (an MFMA kernel loading straight to registers up to 32
// tokens, depth-split 128 x 192 tiles and a reduction pass above), us:
//     tokens x rows of B x depth     before   now
//     13 x  1536 x 11008              20.7   13.1
//     13 x  2458 x  6144              20.7   11.0
//     24 x 12288 x  1536              16.5   11.1
//     48 x  1536 x  4096              18.9    9.9
//     48 x 12288 x  1536              17.1   12.5
//     64 x 22016 x  1536              26.0   20.2
//    128 x  4096 x  1536              18.2    9.3
//    333 x  2458 x  6144              31.6   27.7
//
// SEG = 2 (up to 16 tokens on few rows of B): the 16 rows of an MFMA operand
// are 8 rows x the 2 halves of a step, so that twice as many workgroups share
// the rows of B; of the 16 x 16 result the two blocks whose halves agree are
// the sums, added at the end (the other two are not used; the matrix cores
// are idle here).  1536 x 11008: 11.2 against 13.7 us at 8 tokens, 12.7
// against 15.0 at 13.
//
// The depth can also be split over S workgroups per tile (fp32 partial sums,
// then the reduction kernel), for deep products with few tiles.
//
// Depth tail: 16-byte chunks at or past D are loaded from past the buffer
// (zeros); the chunk that straddles D is masked in registers, both operands.
#include <algorithm>
#include <cmath>

#include "common.hpp"
#include "kernels.hpp"

namespace espace {

namespace {

constexpr int MK = 64;                            // depth of a step: 128-byte rows

// BM, BN, W, ST, SEG: as many waves and stages as 160 KB of LDS hold, eight
// waves for the narrow tiles (more loads in flight), four for the others.
#define MID_CONFIGS(X)                                                                                        \
    X(8, 8, 8, 8, 2) X(16, 8, 8, 6, 2)                                                                        \
    X(16, 16, 8, 4, 1) X(16, 32, 8, 3, 1) X(16, 48, 8, 2, 1) X(16, 64, 4, 4, 1) X(16, 80, 4, 3, 1) X(16, 96, 4, 2, 1) \
    X(32, 16, 8, 3, 1) X(32, 32, 4, 4, 1) X(32, 48, 4, 4, 1) X(32, 64, 4, 3, 1) X(32, 80, 4, 2, 1) X(32, 96, 4, 2, 1) \
    X(48, 16, 8, 2, 1) X(48, 32, 4, 4, 1) X(48, 48, 4, 3, 1) X(48, 64, 4, 2, 1) X(48, 80, 4, 2, 1) X(48, 96, 4, 2, 1) \
    X(64, 16, 8, 2, 1) X(64, 32, 4, 3, 1) X(64, 48, 4, 2, 1) X(64, 64, 4, 2, 1) X(64, 80, 4, 2, 1) X(64, 96, 4, 2, 1) \
    X(80, 32, 4, 2, 1) X(80, 48, 4, 2, 1) X(80, 64, 4, 2, 1) X(80, 80, 4, 2, 1)                               \
    X(96, 32, 4, 2, 1) X(96, 48, 4, 2, 1) X(96, 64, 4, 2, 1) X(112, 48, 4, 2, 1)

struct MidShape { int bm, bn, waves; };
constexpr MidShape kMid[] = {
#define X(BM, BN, W, ST, SEG) {BM, BN, W},
    MID_CONFIGS(X)
#undef X
};
constexpr int kMidCount = sizeof(kMid) / sizeof(kMid[0]);
constexpr int kMidMaxRows = 112;                  // largest BM or BN

template <int BM, int BN, int W, int ST, int SEG>
struct MidCfg {
    static constexpr int ROWS = BM + BN;
    static constexpr int STAGE = ROWS * MK * 2;
    static constexpr int LPS = ROWS / 8;          // 1 KB loads (8 rows) per stage
    static constexpr int GR = 16 / SEG;           // rows of an operand per MFMA
    static constexpr int TM = BM / GR, TN = BN / GR;
    static constexpr int NS = 2 / SEG;            // MFMAs per step and block
    static constexpr int RING = W * ST * STAGE;
    static constexpr int RED = W * TM * TN * 1024;
    static constexpr int SMEM = RING > RED ? RING : RED;
    static_assert(SMEM <= 160 * 1024 && LPS * (ST - 1) < 64, "sizes");
    static_assert(BM % GR == 0 && BN % GR == 0 && BM <= kMidMaxRows && BN <= kMidMaxRows, "tile");
};

// this wave's loads but the newest N have landed; no memory access moves
// across (the loads into LDS are invisible to the compiler)
template <int N>
__device__ __forceinline__ void mid_wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// part != nullptr: depth range blockIdx.y (`sps` steps) as fp32 sums at part +
// blockIdx.y * split_stride, leading dimension ldp; else C in bf16.
template <int BM, int BN, int W, int ST, int SEG>
__global__ __launch_bounds__(W * 64, W / 4)
void mid_tn_bf16_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B, int64_t ldb,
                        uint16_t* __restrict__ C, int64_t ldc, int R, int Cc, int D, int tiles_c, int c_pairs,
                        float* __restrict__ part, int64_t ldp, int64_t split_stride, int sps, int upper) {
    using T = MidCfg<BM, BN, W, ST, SEG>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[T::SMEM];
    int tile_r, tile_c;
    tile_coords<8>(blockIdx.x, gridDim.x, tiles_c, 0, tile_r, tile_c);
    const int row0 = tile_r * BM, col0 = tile_c * BN;
    // a symmetric product: nothing of the tile lies in a 32 x 32 block on or above
    // the diagonal
    if (upper && row0 / 32 > (col0 + BN - 1) / 32) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char* ring = smem + wave * ST * T::STAGE;

    // descriptors over the tile's own rows (fewer than 2^31 bytes, the
    // launcher checks); rows past the matrix repeat its last row
    const int nr = min(BM, R - row0), nc = min(BN, Cc - col0);
    const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (int64_t)row0 * lda), (short)0,
                                                      (int)((uint64_t)nr * lda * 2u), 0x00020000);
    const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)(B + (int64_t)col0 * ldb), (short)0,
                                                      (int)((uint64_t)nc * ldb * 2u), 0x00020000);
    // load j covers rows 8 j .. 8 j + 7 of the tile's token rows, then rows of
    // B; chunk c of row r sits at chunk c ^ ((r >> 1) & 7), so that the rows
    // one fragment read touches fall on distinct banks
    unsigned off[T::LPS];
#pragma unroll
    for (int j = 0; j < T::LPS; ++j) {
        const bool isA = 8 * j < BM;
        const int rr = 8 * j + (lane >> 3) - (isA ? 0 : BM);
        const int c = (lane & 7) ^ ((rr >> 1) & 7);
        off[j] = ((unsigned)(isA ? min(rr, nr - 1) : min(rr, nc - 1)) * (unsigned)(isA ? lda : ldb) + c * 8) * 2u;
    }
    const int steps = (D + MK - 1) / MK;
    const int s0 = blockIdx.y * sps;
    const int ns = min(sps, steps - s0);          // steps of this depth range
    const int mine = ns > wave ? (ns - wave + W - 1) / W : 0;   // of this wave: s0 + wave, s0 + wave + W, ...
    const DepthOrder order(0, ns > 0 ? ns : 0);   // the XCDs start at different depths
    // the loads of this wave's step t into stage st; past the depth they are
    // still issued, reading past the buffers, so that the count of loads in
    // flight is the same throughout
    auto issue = [&](int t, int st) {
        unsigned char* stage = ring + st * T::STAGE;
        const int k0 = (s0 + order(t * W + wave)) * MK;
        if (k0 + MK <= D) {
#pragma unroll
            for (int j = 0; j < T::LPS; ++j)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(8 * j < BM ? ra : rb,
                                                         (__attribute__((address_space(3))) void*)(stage + j * 1024),
                                                         16, (int)off[j], k0 * 2, 0, 0);
        } else {
#pragma unroll
            for (int j = 0; j < T::LPS; ++j) {
                const int rr = 8 * j + (lane >> 3) - (8 * j < BM ? 0 : BM);
                const int k = k0 + 8 * ((lane & 7) ^ ((rr >> 1) & 7));
                const unsigned o = k < D ? off[j] + (unsigned)k0 * 2u : 0x7FFFFFF0u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(8 * j < BM ? ra : rb,
                                                         (__attribute__((address_space(3))) void*)(stage + j * 1024),
                                                         16, (int)o, 0, 0, 0);
            }
        }
    };

    f32x4_t acc[T::TM][T::TN];
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // fragment row of this lane, its first chunk, and (SEG = 2) its half of the step
    const int lr = lane & (T::GR - 1), lq = lane >> 4;
    const int seg = SEG == 2 ? (lane >> 3) & 1 : 0;
    // byte offset of chunk 4 (s + seg) + lq of the lane's row of block i
    auto at = [&](int i, int s) {
        const int r = T::GR * i + lr;
        return r * 128 + (((4 * (s + seg) + lq) ^ ((r >> 1) & 7)) << 4);
    };

#pragma unroll
    for (int p = 0; p < ST; ++p) issue(p, p);
    int st = 0;
    for (int t = 0; t < mine; ++t) {
        mid_wait_vm<(ST - 1) * T::LPS>();
        const unsigned char* pa = ring + st * T::STAGE;
        const unsigned char* pb = pa + BM * 128;
        u32x4_t fa[T::NS][T::TM], fb[T::NS][T::TN];
#pragma unroll
        for (int s = 0; s < T::NS; ++s) {
#pragma unroll
            for (int i = 0; i < T::TM; ++i) fa[s][i] = *reinterpret_cast<const u32x4_t*>(pa + at(i, s));
#pragma unroll
            for (int j = 0; j < T::TN; ++j) fb[s][j] = *reinterpret_cast<const u32x4_t*>(pb + at(j, s));
        }
        const int left = D - (s0 + order(t * W + wave)) * MK;
        if (left < MK) {
#pragma unroll
            for (int s = 0; s < T::NS; ++s) {
                const int nv = left - 32 * (s + seg) - 8 * lq;
                const int v = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
#pragma unroll
                for (int i = 0; i < T::TM; ++i) fa[s][i] = mask_chunk(fa[s][i], v);
#pragma unroll
                for (int j = 0; j < T::TN; ++j) fb[s][j] = mask_chunk(fb[s][j], v);
            }
        }
        // this wave is done reading the stage: it receives step t + ST
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(t + ST, st);
        st = st + 1 == ST ? 0 : st + 1;
#pragma unroll
        for (int s = 0; s < T::NS; ++s)
#pragma unroll
            for (int i = 0; i < T::TM; ++i)
#pragma unroll
                for (int j = 0; j < T::TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fb[s][j]), as_bf16x8(fa[s][i]),
                                                                        acc[i][j], 0, 0, 0);
    }
    // every load into LDS has landed (those past the depth wrote zeros)
    // before the sums take the rings' place
    mid_wait_vm<0>();
    __syncthreads();
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);
    constexpr int NB = T::TM * T::TN;
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j) red[(wave * NB + i * T::TN + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    // lane l of a block holds token l % 16, columns 4 (l / 16) .. + 3 (SEG = 2:
    // token l % 8 of half (l / 8) % 2; columns 0..7 of half 0 in lanes 0..31,
    // of half 1 in lanes 32..63, so the other half's sum is in lane l ^ 40)
    for (int b = wave; b < NB; b += W) {
        f32x4_t v = red[b * 64 + lane];
#pragma unroll
        for (int w = 1; w < W; ++w) v += red[(w * NB + b) * 64 + lane];
        if constexpr (SEG == 2) {
#pragma unroll
            for (int w = 0; w < W; ++w) v += red[(w * NB + b) * 64 + (lane ^ 40)];
        }
        const int r = row0 + T::GR * (b / T::TN) + lr;
        const int c = col0 + T::GR * (b % T::TN) + 4 * lq;
        if (r >= R || c >= Cc || (SEG == 2 && (seg || lane >= 32))) continue;
        if (part) {
            // ldp is a multiple of 8: the run of 4 stays inside the row
            *reinterpret_cast<f32x4_t*>(part + blockIdx.y * split_stride + (int64_t)r * ldp + c) = v;
            continue;
        }
        // c is a multiple of 4: the run stays inside one 32-column block of
        // the row-pair layout
        uint16_t* p = C + (c_pairs ? pair_offset(r, c, ldc) : (int64_t)r * ldc + c);
        if (c + 4 <= Cc) {
            *reinterpret_cast<u32x2_t*>(p) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c + e < Cc) p[e] = (uint16_t)bf16_rne(v[e]);
        }
    }
}

template <int BM, int BN, int W, int ST, int SEG>
hipError_t launch_cfg_mid(const GemmArgs& g, bool upper, hipStream_t stream) {
    const int tr = (g.R + BM - 1) / BM, tc = (g.Cc + BN - 1) / BN;
    const int steps = (g.D + MK - 1) / MK;
    const int S = g.splits > 1 ? g.splits : 1;
    const int64_t ldp = splitk_ld(g.Cc), stride = (int64_t)g.R * ldp;
    hipLaunchKernelGGL((mid_tn_bf16_kernel<BM, BN, W, ST, SEG>), dim3(tr * tc, S), dim3(W * 64), 0, stream, g.A,
                       g.lda, g.B, g.ldb, (uint16_t*)g.C, g.ldc, g.R, g.Cc, g.D, tc, g.c_pairs,
                       S > 1 || upper ? g.partial : nullptr, ldp, stride, (steps + S - 1) / S, upper ? 1 : 0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1 || upper) return e;
    return launch_splitk_reduce(g.partial, S, stride, ldp, g.C, g.ldc, g.R, g.Cc, g.c_pairs ? 2 : 1, stream);
}

}  // namespace

// Estimated time of a product (us) with the best of the tiles, from what
// bounds it: B from HBM at 5.3 TB/s and the tiles' operand bytes through each
// CU's load path at 74 KB/us, round by round, which overlap to the root of their
// squares' sum.  Rows off the cache lines cost 25% of the one and 34% of the other,
// half lines a third of that (a step's 128 bytes of a row are two lines),
// half-filled operands 5% of the other.  A launch is 2.85 us, each further round 2.7
// (the rings drain and refill; one workgroup fits a CU), a depth split the reduction
// launch and its traffic.  Fitted with the tiled kernels' price (espace_api.hip), to
// 2800 times of these tiles at 3 to 1024 tokens.
double mid_plan(int R, int Cc, int D, int cus, int ranges, int* config, int* splits) {
    double best = 1e300;
    const int steps = (D + MK - 1) / MK;
    const int64_t row_bytes = ((int64_t)D + 7) / 8 * 16;
    const double off_line = row_bytes % 128 == 0 ? 0.0 : (row_bytes % 64 == 0 ? 0.33 : 1.0);
    const double hbm = 2e-6 * Cc * D / 5.32 * (1.0 + 0.25 * off_line);
    for (int i = 0; i < kMidCount; ++i) {
        const int bm = kMid[i].bm, bn = kMid[i].bn;
        // half-filled operands serve only token counts that fit one tile
        if (bn == 8 && R > bm) continue;
        if (bm >= 16 && bm - 16 >= R) continue;    // a smaller tile holds all tokens
        const int64_t tiles = (int64_t)((R + bm - 1) / bm) * ((Cc + bn - 1) / bn);
        for (int s = 1; s <= ranges; ++s) {
            if (s > 1 && steps / s < 32) break;    // at least 4 to 8 steps per wave
            // up to 16 tokens: only where the tiles leave most CUs idle (512 x 24576 at
            // one token 14.2 -> 10.8 us with four ranges, but 6144 x 24576 54 -> 60, at 8
            // tokens 57 -> 60)
            if (s > 1 && R <= 16 && Cc > 10 * cus) break;
            const int64_t rounds = (tiles * s + cus - 1) / cus;
            const double load = rounds * (bm + bn) * (double)((steps + s - 1) / s) * (MK * 2) / 74e3 *
                                (1.0 + 0.34 * off_line) * (bn == 8 ? 1.05 : 1.0);
            double t = 2.85 + std::sqrt(hbm * hbm + load * load) + 2.7 * (rounds - 1) + 0.0004 * bm * bn;
            if (s > 1) t += 3.4 + 1.3e-6 * s * R * (double)Cc;
            if (t < best) {
                best = t;
                *config = i;
                *splits = s;
            }
        }
    }
    return best;
}

int mid_waves(int config) { return kMid[config].waves; }

// The tiles' 32-bit offsets.
bool mid_supported(int64_t lda, int64_t ldb) {
    return std::max(lda, ldb) * kMidMaxRows * 2 < ((int64_t)1 << 31);
}

static hipError_t launch_config(const GemmArgs& g, bool upper, hipStream_t stream) {
    int i = 0;
#define X(BM, BN, W, ST, SEG) \
    if (g.tile == i++) return launch_cfg_mid<BM, BN, W, ST, SEG>(g, upper, stream);
    MID_CONFIGS(X)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_mid_tn_bf16(const GemmArgs& g, hipStream_t stream) {
    if (!mid_supported(g.lda, g.ldb) || g.a_pairs || g.c_f32) return hipErrorInvalidValue;
    return launch_config(g, false, stream);
}

hipError_t launch_mid_tn_bf16_ranges(const GemmArgs& g, hipStream_t stream) {
    if (!mid_supported(g.lda, g.ldb) || g.R != g.Cc || !g.partial) return hipErrorInvalidValue;
    return launch_config(g, true, stream);
}

}  // namespace espace
