// Tiled bfloat16 "TN" GEMM whose waves split the tile and every depth step:
//
//     C[r][c] = sum_k A[r][k] * B[c][k]        (fp32 accumulation)
//
// Eight waves, two per SIMD, as 2 x 2 over the tile and 2 over the depth: of
// every 64-deep step the waves of half h take the 32 of chunks 4 h .. 4 h + 3
// for their quarter of the tile (v_mfma_f32_16x16x32_bf16).  Against eight
// waves spread over the tile a step reads far fewer fragment bytes from LDS
// (128 x 192: 80 KB instead of 128, which with the 40 KB written bounded the
// kernel of gemm_bf16_v2.hip); rows are 128 bytes, one request per cache line
// (the four-wave kernel of gemm_bf16_v3.hip makes two).  One barrier per step.
// The halves' sums are added through LDS at the end, each wave finishing every
// other block.  Operands rotated through HBM, us, the best of the other
// kernels -> this one:
//  * 128 x 192, long depths (one round of 256 tiles on the Llama2-7B
//    projections): four LDS stages (all 160 KB), one step of fragments read
//    ahead.  4096 x 1536 x 4096 57 -> 56, x 11008 158 -> 134, x 12288 162 -> 145.
//    Bound by the operands through each CU's load path: the same loads without
//    arithmetic take 48 of the 55 at depth 4096, the arithmetic alone 40, the
//    LDS reads alone 22 (10 of each are launch, ramp and writing the tile).
//    Three stages: 2 more.  Below about 48 steps the sums' exchange costs more
//    than the loop gains (512 x 12288 x 1536: 27.0 against 25.2).
//  * 192 x 192 and 256 x 160, where they fill the chip's rounds better than
//    256 x 256, 256 x 192 or 128 x 192: too many accumulators for reading
//    ahead, so the two halves alternate between reading and multiplying.  512 tiles
//    of 192 x 192: 12288 x 1536 x 4096 146 (256 x 192) -> 142, in the training step,
//    its operands partly in the cache, 158 (two launches by rows) -> 152; 512 of 256 x
//    160: 8192 x 2458 x 24576 982 -> 837 (two launches by rows: 800); 333 x 24576 x 2458
//    71 -> 57 on 192 x 192.  At equal rounds the four-wave kernel's larger tiles are
//    10 to 25% faster.
#include "common.hpp"
#include "kernels.hpp"

namespace espace {

namespace {

constexpr int DK = 64;                            // depth of a step: 128-byte rows

template <int BM, int BN, int ST>
struct DCfg {
    static constexpr int ROWS = BM + BN;
    static constexpr int STAGE = ROWS * DK * 2;
    static constexpr int NLOAD = ROWS / 8;
    static constexpr int LPW = (NLOAD + 7) / 8;   // 1 KB loads per wave and stage (uniform: extra ones repeat a load)
    static constexpr int TM = BM / 32, TN = BN / 32;
    static constexpr int NB = TM * TN;
    static constexpr int RED = 8 * ((NB + 1) / 2) * 1024;
    static constexpr int SMEM = ST * STAGE > RED ? ST * STAGE : RED;
    static_assert(SMEM <= 160 * 1024 && LPW * ST < 64 && BM % 32 == 0 && BN % 32 == 0, "sizes");
};

template <int N>
__device__ __forceinline__ void d_wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void d_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// part != nullptr: depth range blockIdx.y (`sps` steps) as fp32 sums at part +
// blockIdx.y * split_stride, leading dimension ldp; else C in bf16, c_pairs in
// the row-pair layout.
template <int BM, int BN, int ST, bool AHEAD>
__global__ __launch_bounds__(512, 2)
void gemm_tn_bf16_v4_kernel(const uint16_t* __restrict__ A, int64_t lda, const uint16_t* __restrict__ B, int64_t ldb,
                            uint16_t* __restrict__ C, int64_t ldc, int R, int Cc, int D, int tiles_c, int c_pairs,
                            float* __restrict__ part, int64_t ldp, int64_t split_stride, int sps) {
    using T = DCfg<BM, BN, ST>;
    constexpr int TM = T::TM, TN = T::TN;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[T::SMEM];
    int tile_r, tile_c;
    tile_coords<4>(blockIdx.x, gridDim.x, tiles_c, 0, tile_r, tile_c);
    const int row0 = tile_r * BM, col0 = tile_c * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave >> 2;                   // depth half of every step
    const int wr0 = ((wave >> 1) & 1) * (BM / 2), wc0 = (wave & 1) * (BN / 2);

    // fewer than 2^31 elements each (the launcher checks): 32-bit byte offsets
    const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)A, (short)0, (int)(uint32_t)((uint64_t)R * lda * 2u),
                                                      0x00020000);
    const auto rb = __builtin_amdgcn_make_buffer_rsrc((void*)B, (short)0, (int)(uint32_t)((uint64_t)Cc * ldb * 2u),
                                                      0x00020000);
    // load j of this wave covers rows 8 q .. 8 q + 7 of the A|B tile, q = wave +
    // 8 j; chunk c of row r sits at chunk c ^ ((r >> 1) & 7)
    unsigned off[T::LPW];
#pragma unroll
    for (int j = 0; j < T::LPW; ++j) {
        const int q = min(wave + 8 * j, T::NLOAD - 1);
        const bool isA = 8 * q < BM;
        const int rr = 8 * q + (lane >> 3) - (isA ? 0 : BM);
        const int c = (lane & 7) ^ ((rr >> 1) & 7);
        const int g = isA ? min(row0 + rr, R - 1) : min(col0 + rr, Cc - 1);
        off[j] = ((unsigned)g * (unsigned)(isA ? lda : ldb) + c * 8) * 2u;
    }
    const int ktiles = (D + DK - 1) / DK;
    const int kt0 = blockIdx.y * sps;
    const int kt_end = min(kt0 + sps, ktiles);
    const DepthOrder order(kt0, BM == 192 ? kt0 : kt_end);
    // loads of step kt into stage st; past the range they still are issued, from
    // past the buffers, so that the count in flight is the same throughout;
    // chunks past the depth are zeros, the one that straddles it is masked
    // before use
    auto issue = [&](int kt, int st) {
        unsigned char* stage = smem + st * T::STAGE;
        const int k0 = order(kt) * DK;
        if (k0 + DK <= D && kt < kt_end) {
#pragma unroll
            for (int j = 0; j < T::LPW; ++j) {
                const int q = min(wave + 8 * j, T::NLOAD - 1);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(8 * q < BM ? ra : rb,
                                                         (__attribute__((address_space(3))) void*)(stage + q * 1024), 16,
                                                         (int)off[j], k0 * 2, 0, 0);
            }
        } else {
#pragma unroll
            for (int j = 0; j < T::LPW; ++j) {
                const int q = min(wave + 8 * j, T::NLOAD - 1);
                const int rr = 8 * q + (lane >> 3) - (8 * q < BM ? 0 : BM);
                const int k = k0 + 8 * ((lane & 7) ^ ((rr >> 1) & 7));
                const unsigned o = k < D && kt < kt_end ? off[j] + (unsigned)k0 * 2u : 0xFFFFFFF0u;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(8 * q < BM ? ra : rb,
                                                         (__attribute__((address_space(3))) void*)(stage + q * 1024), 16,
                                                         (int)o, 0, 0, 0);
            }
        }
    };
    const int lr = lane & 15, lq = lane >> 4;
    const int slot = ((4 * half + lq) ^ ((lr >> 1) & 7)) << 4;
    const int a_off = (wr0 + lr) * 128 + slot, b_off = (BM + wc0 + lr) * 128 + slot;

    f32x4_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    constexpr int NF = AHEAD ? 2 : 1;             // fragment buffers
    u32x4_t fa[NF][TM], fb[NF][TN];
    auto read = [&](int buf, int st) {
        const unsigned char* s = smem + st * T::STAGE;
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[buf][j] = *reinterpret_cast<const u32x4_t*>(s + b_off + j * 2048);
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[buf][i] = *reinterpret_cast<const u32x4_t*>(s + a_off + i * 2048);
    };
    auto mfmas = [&](int buf, int kt) {
        const int left = D - order(kt) * DK;
        if (left < DK) {
            const int nv = left - 32 * half - 8 * lq;
            const int v = nv < 0 ? 0 : (nv > 8 ? 8 : nv);
#pragma unroll
            for (int i = 0; i < TM; ++i) fa[buf][i] = mask_chunk(fa[buf][i], v);
#pragma unroll
            for (int j = 0; j < TN; ++j) fb[buf][j] = mask_chunk(fb[buf][j], v);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(fb[buf][j]), as_bf16x8(fa[buf][i]),
                                                                    acc[i][j], 0, 0, 0);
    };
    int st = 0;
    if constexpr (AHEAD) {
        // stages hold steps kt .. kt + ST - 1; one step of fragments is read ahead
#pragma unroll
        for (int p = 0; p < ST; ++p) issue(kt0 + p, p);
        d_wait_vm<(ST - 1) * T::LPW>();
        d_barrier();
        read(0, 0);
        auto step = [&](int buf, int kt) {
            // this wave's loads of step kt + 1 have landed; after the barrier
            // every wave's, and every wave has its fragments of step kt: its
            // stage is free
            d_wait_vm<(ST - 2) * T::LPW>();
            d_barrier();
            issue(kt + ST, st);
            st = st + 1 == ST ? 0 : st + 1;
            read(buf ^ 1, st);
            mfmas(buf, kt);
        };
        int kt = kt0;
        for (; kt + 1 < kt_end; kt += 2) {
            step(0, kt);
            step(1, kt + 1);
        }
        if (kt < kt_end) step(0, kt);
    } else {
        // one fragment buffer: the waves of the first half read a step, then
        // multiply it; those of the second multiply the step before while the
        // others read, then read theirs
#pragma unroll
        for (int p = 0; p < ST - 1; ++p) issue(kt0 + p, p);
        auto phase = [&](int kt) {
            // step kt has landed for this wave, after the barrier for all, and
            // every wave is done reading step kt - 1, whose stage is refilled
            d_wait_vm<(ST - 2) * T::LPW>();
            d_barrier();
            issue(kt + ST - 1, st == 0 ? ST - 1 : st - 1);
        };
        if (half == 0) {
            for (int kt = kt0; kt < kt_end; ++kt) {
                phase(kt);
                read(0, st);
                st = st + 1 == ST ? 0 : st + 1;
                mfmas(0, kt);
            }
        } else {
            for (int kt = kt0; kt < kt_end; ++kt) {
                phase(kt);
                if (kt > kt0) mfmas(0, kt - 1);
                read(0, st);
                st = st + 1 == ST ? 0 : st + 1;
            }
            if (kt_end > kt0) mfmas(0, kt_end - 1);
        }
    }
    d_wait_vm<0>();
    __syncthreads();

    // ---- the two depth halves: each wave finishes every other block and hands
    // the others to the wave of the other half
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);
    constexpr int HB = (T::NB + 1) / 2;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int b = i * TN + j;
            if ((b & 1) != half) red[((wave ^ 4) * HB + (b >> 1)) * 64 + lane] = acc[i][j];
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int b = i * TN + j;
            if ((b & 1) != half) continue;
            const f32x4_t v = acc[i][j] + red[(wave * HB + (b >> 1)) * 64 + lane];
            const int r = row0 + wr0 + 16 * i + lr;
            const int c = col0 + wc0 + 16 * j + 4 * lq;
            if (r >= R || c >= Cc) continue;
            if (part) {
                *reinterpret_cast<f32x4_t*>(part + blockIdx.y * split_stride + (int64_t)r * ldp + c) = v;
                continue;
            }
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

template <int BM, int BN, int ST, bool AHEAD>
hipError_t launch_cfg_v4(const GemmArgs& g, hipStream_t stream) {
    const int tr = (g.R + BM - 1) / BM, tc = (g.Cc + BN - 1) / BN;
    const int steps = (g.D + DK - 1) / DK;
    const int S = g.splits > 1 ? g.splits : 1;
    const int64_t ldp = splitk_ld(g.Cc), stride = (int64_t)g.R * ldp;
    hipLaunchKernelGGL((gemm_tn_bf16_v4_kernel<BM, BN, ST, AHEAD>), dim3(tr * tc, S), dim3(512), 0, stream, g.A, g.lda, g.B,
                       g.ldb, (uint16_t*)g.C, g.ldc, g.R, g.Cc, g.D, tc, g.c_pairs, S > 1 ? g.partial : nullptr, ldp,
                       stride, (steps + S - 1) / S);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || S == 1) return e;
    return launch_splitk_reduce(g.partial, S, stride, ldp, g.C, g.ldc, g.R, g.Cc, g.c_pairs ? 2 : 1, stream);
}

}  // namespace

hipError_t launch_gemm_tn_bf16_v4(const GemmArgs& g, hipStream_t stream) {
    const int64_t lim = (int64_t)1 << 31;
    if ((int64_t)g.R * g.lda >= lim || (int64_t)g.Cc * g.ldb >= lim || g.a_pairs || g.pair || g.c_f32)
        return hipErrorInvalidValue;
    switch (g.tile) {
        case TILE_128x192: return launch_cfg_v4<128, 192, 4, true>(g, stream);
        case TILE_192x192: return launch_cfg_v4<192, 192, 3, false>(g, stream);
        case TILE_256x160: return launch_cfg_v4<256, 160, 3, false>(g, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace espace
