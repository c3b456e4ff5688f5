// MX-FP8 products out[r][c] = sum_d T[r][d] * W[c][d] for up to a thousand
// tokens: the small-tile kernel of the bfloat16 product (mid_bf16.hip) on
// block-scaled operands.  A step is 128 codes deep, 128 bytes per row as
// there, and one v_mfma_scale_f32_16x16x128_f8f6f4 per 16 x 16 block (operand
// layout: gemm_mxfp8.hip); the waves split the depth, each with its own ring
// of LDS stages, and their sums are added in wave order, so a sum's chain in
// the limited-precision accumulation of that instruction is shorter than a
// tiled kernel's.
//
// The scale bytes of the tile's rows are brought into LDS whole, once, while
// the first stages are in flight (a row's scales are 1/32 of its codes): for
// four steps at a time 16 bytes per row, [four steps][row], so that the byte
// reads of 16 rows fall on distinct banks; 4 bytes per row and step where the
// scale rows do not start on 16 bytes.  The LDS the ring leaves bounds the
// depth a configuration takes (fits).
//
// Priced by the operands through each CU's load path, 70 KB/us, or the weight
// from HBM; at the sizes below launch, ramp and the final sums weigh as much (48 x
// 1536 x 11008: data return busy 30% of the time, L2 60%).  Measured with operands rotated through HBM, us, against one
// 128 x 128 or 256 x 128 tile per workgroup (a few dozen workgroups):
//     projection   8 x 1536 x  4096   24.1 ->  6.6
//     projection  48 x 1536 x 11008   71.7 -> 13.2
//     projection 333 x 2458 x  6144   43.7 -> 17.7
//     expansion    8 x 22016 x 1536   13.8 -> 10.0
//     expansion   64 x 12288 x 1536   14.6 ->  9.3
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"
#include "mx_core.hpp"

namespace espace {

namespace {

constexpr int MXK = 128;                          // depth of a step: 128-byte rows

// BM, BN, W, ST
#define MXMID_CONFIGS(X)                                                              \
    X(16, 16, 8, 4) X(16, 32, 8, 2) X(16, 48, 8, 2) X(16, 64, 4, 3) X(16, 96, 4, 2)   \
    X(32, 16, 8, 2) X(32, 32, 4, 3) X(32, 48, 4, 3) X(32, 64, 4, 2) X(32, 96, 4, 2)   \
    X(48, 16, 8, 2) X(48, 32, 4, 2) X(48, 48, 4, 2) X(48, 64, 4, 2) X(48, 80, 4, 2) X(48, 96, 4, 2) \
    X(64, 32, 4, 2) X(64, 48, 4, 2) X(64, 64, 4, 2) X(64, 80, 4, 2)                   \
    X(80, 48, 4, 2) X(80, 64, 4, 2) X(96, 32, 4, 2) X(96, 48, 4, 2)

template <int BM, int BN, int W, int ST>
struct MxMidCfg {
    static constexpr int ROWS = BM + BN;
    static constexpr int STAGE = ROWS * MXK;
    static constexpr int LPS = ROWS / 8;
    static constexpr int TM = BM / 16, TN = BN / 16;
    static constexpr int RING = W * ST * STAGE;
    static constexpr int SCALES = 160 * 1024 - RING;
    static constexpr int SMEM = RING + SCALES;
    static_assert(W * TM * TN * 1024 <= SMEM && SCALES >= 8 * 1024 && LPS * ST < 64, "sizes");
    static constexpr bool fits(int D) { return ((D + 511) / 512) * ROWS * 16 <= SCALES; }
};

template <int N>
__device__ __forceinline__ void mxmid_wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int BM, int BN, int W, int ST, int SS, int ZOUT>
__global__ __launch_bounds__(W * 64, W / 4)
void mid_mx_kernel(MxGemmArgs a, int tiles_c) {
    using T = MxMidCfg<BM, BN, W, ST>;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[T::SMEM];
    int tile_r, tile_c;
    tile_coords<8>(blockIdx.x, gridDim.x, tiles_c, 0, tile_r, tile_c);
    const int row0 = tile_r * BM, col0 = tile_c * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    unsigned char* ring = smem + wave * ST * T::STAGE;
    unsigned char* scales = smem + T::RING;

    // a tile past the last column (MX-FP8 output up to cpad) reads the last row of W
    const int cb0 = min(col0, a.C - 1);
    const int nr = min(BM, a.R - row0), nc = min(BN, a.C - cb0);
    const auto rt = __builtin_amdgcn_make_buffer_rsrc((void*)(a.T + (int64_t)row0 * a.ldt), (short)0,
                                                      (int)(nr * a.ldt), 0x00020000);
    const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)(a.W + (int64_t)cb0 * a.ldw), (short)0,
                                                      (int)(nc * a.ldw), 0x00020000);
    const auto rts = __builtin_amdgcn_make_buffer_rsrc((void*)(a.Ts + (int64_t)row0 * a.ldts), (short)0,
                                                       (int)(nr * a.ldts), 0x00020000);
    const auto rws = __builtin_amdgcn_make_buffer_rsrc((void*)(a.Ws + (int64_t)cb0 * a.ldws), (short)0,
                                                       (int)(nc * a.ldws), 0x00020000);
    const int steps = (a.D + MXK - 1) / MXK;
    const int mine = steps > wave ? (steps - wave + W - 1) / W : 0;

    unsigned off[T::LPS];
#pragma unroll
    for (int j = 0; j < T::LPS; ++j) {
        const bool isT = 8 * j < BM;
        const int rr = 8 * j + (lane >> 3) - (isT ? 0 : BM);
        const int c = (lane & 7) ^ ((rr >> 1) & 7);
        off[j] = (unsigned)(isT ? min(rr, nr - 1) : min(rr, nc - 1)) * (unsigned)(isT ? a.ldt : a.ldw) + c * 16;
    }
    // the loads of this wave's step t into stage st; past the last step they
    // are still issued, so that the count of loads in flight is the same
    auto issue = [&](int t, int st) {
        unsigned char* stage = ring + st * T::STAGE;
        const int s = t * W + wave;
        const int k0 = s < steps ? s * MXK : 0;
        const unsigned past = s < steps ? 0u : 0x80000000u;   // past the buffers: zeros, no traffic
#pragma unroll
        for (int j = 0; j < T::LPS; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(8 * j < BM ? rt : rw,
                                                     (__attribute__((address_space(3))) void*)(stage + j * 1024), 16,
                                                     (int)(off[j] | past), k0, 0, 0);
    };

    f32x4_t acc[T::TM][T::TN];
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int lr = lane & 15, lq = lane >> 4, sw = (lr >> 1) & 7;
#pragma unroll
    for (int p = 0; p < ST; ++p) issue(p, p);
    // the tile's scale bytes, [group of SS steps][row]
    {
        const int total = ((steps + SS - 1) / SS) * T::ROWS;
        for (int p0 = wave * 64; p0 < total; p0 += W * 64) {
            const int p = p0 + lane;
            const int g = p / T::ROWS, r = p - g * T::ROWS;
            const bool tok = r < BM;
            const int rr = tok ? min(r, nr - 1) : min(r - BM, nc - 1);
            const unsigned o = (unsigned)rr * (unsigned)(tok ? a.ldts : a.ldws) + g * (4 * SS);
            if constexpr (SS == 4) {
                // a last group may read past the matrix's steps (bytes not
                // used; past the buffer they are zeros)
                if (p < total) {
                    const auto x = tok ? __builtin_amdgcn_raw_buffer_load_b128(rts, (int)o, 0, 0)
                                       : __builtin_amdgcn_raw_buffer_load_b128(rws, (int)o, 0, 0);
                    *reinterpret_cast<u32x4_t*>(scales + p * 16) = u32x4_t{x[0], x[1], x[2], x[3]};
                }
            } else {
                if (p < total) {
                    const uint32_t x = tok ? __builtin_amdgcn_raw_buffer_load_b32(rts, (int)o, 0, 0)
                                           : __builtin_amdgcn_raw_buffer_load_b32(rws, (int)o, 0, 0);
                    *reinterpret_cast<uint32_t*>(scales + p * 4) = x;
                }
            }
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wave's scales are in LDS
    int st = 0;
    for (int t = 0; t < mine; ++t) {
        mxmid_wait_vm<(ST - 1) * T::LPS>();
        const unsigned char* pt = ring + st * T::STAGE + lr * MXK;
        const unsigned char* pw = pt + BM * MXK;
        const int s = t * W + wave;
        const unsigned char* sc = scales + (SS == 4 ? ((s >> 2) * T::ROWS + lr) * 16 + (s & 3) * 4 : (s * T::ROWS + lr) * 4) + lq;
        i32x8_t ft[T::TM], fw[T::TN];
        int st_[T::TM], sw_[T::TN];
        auto frag = [&](const unsigned char* p) {
            const i32x4_t lo = *reinterpret_cast<const i32x4_t*>(p + ((lq ^ sw) << 4));
            const i32x4_t hi = *reinterpret_cast<const i32x4_t*>(p + (((4 + lq) ^ sw) << 4));
            return i32x8_t{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        };
#pragma unroll
        for (int i = 0; i < T::TM; ++i) {
            ft[i] = frag(pt + i * 16 * MXK);
            st_[i] = sc[i * 16 * 4 * SS];
        }
#pragma unroll
        for (int j = 0; j < T::TN; ++j) {
            fw[j] = frag(pw + j * 16 * MXK);
            sw_[j] = sc[(BM + j * 16) * 4 * SS];
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(t + ST, st);
        st = st + 1 == ST ? 0 : st + 1;
#pragma unroll
        for (int i = 0; i < T::TM; ++i)
#pragma unroll
            for (int j = 0; j < T::TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fw[j], ft[i], acc[i][j], 0, 0, 0, sw_[j], 0,
                                                                            st_[i]);
    }
    mxmid_wait_vm<0>();
    __syncthreads();
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);
    constexpr int NB = T::TM * T::TN;
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j) red[(wave * NB + i * T::TN + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    auto sum = [&](int b) {
        f32x4_t v = red[b * 64 + lane];
#pragma unroll
        for (int w = 1; w < W; ++w) v += red[(w * NB + b) * 64 + lane];
        return v;
    };
    if constexpr (ZOUT) {
        uint8_t* Zq = static_cast<uint8_t*>(a.out);
        for (int b = wave; b < NB / 2; b += W) {
            const f32x4_t x = sum(2 * b), y = sum(2 * b + 1);
            const int n = row0 + 16 * (2 * b / T::TN) + lr;
            const int cb = col0 + 16 * (2 * b % T::TN);      // first column of the 32-column block
            float v[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = (cb + 4 * lq + e < a.C) ? x[e] : 0.f;
                v[4 + e] = (cb + 16 + 4 * lq + e < a.C) ? y[e] : 0.f;
            }
            float amax = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(v[e]));
            amax = fmaxf(amax, __shfl_xor(amax, 16));
            amax = fmaxf(amax, __shfl_xor(amax, 32));
            const int sb = mx_scale_byte(amax);
            const int nsh = 127 - sb;
            if (n < a.R && cb < a.cpad) {
                const int c = cb + 4 * lq;
                uint8_t* p = Zq + (a.out_pairs ? (int64_t)(n >> 1) * a.ldo + (c >> 6) * 128 + (n & 1) * 64 + (c & 63)
                                               : (int64_t)n * a.ldo + c);
                *reinterpret_cast<uint32_t*>(p) =
                    mx_pack4(__builtin_amdgcn_ldexpf(v[0], nsh), __builtin_amdgcn_ldexpf(v[1], nsh),
                             __builtin_amdgcn_ldexpf(v[2], nsh), __builtin_amdgcn_ldexpf(v[3], nsh));
                *reinterpret_cast<uint32_t*>(p + 16) =
                    mx_pack4(__builtin_amdgcn_ldexpf(v[4], nsh), __builtin_amdgcn_ldexpf(v[5], nsh),
                             __builtin_amdgcn_ldexpf(v[6], nsh), __builtin_amdgcn_ldexpf(v[7], nsh));
                if (lq == 0) a.outs[(int64_t)n * a.ldos + cb / 32] = (uint8_t)sb;
            }
        }
    } else {
        uint16_t* Y = static_cast<uint16_t*>(a.out);
        for (int b = wave; b < NB; b += W) {
            const f32x4_t v = sum(b);
            const int r = row0 + 16 * (b / T::TN) + lr;
            const int c = col0 + 16 * (b % T::TN) + 4 * lq;
            if (r >= a.R || c >= a.C) continue;
            uint16_t* p = Y + (int64_t)r * a.ldo + c;
            if (c + 4 <= a.C) {
                *reinterpret_cast<u32x2_t*>(p) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < a.C) p[e] = (uint16_t)bf16_rne(v[e]);
            }
        }
    }
}

template <int BM, int BN, int W, int ST>
hipError_t launch_mx_mid_cfg(const MxGemmArgs& a, int out_mx, bool s16, hipStream_t stream) {
    const int tc = ((out_mx ? a.cpad : a.C) + BN - 1) / BN;
    const dim3 grid(((a.R + BM - 1) / BM) * tc), block(W * 64);
    if (!MxMidCfg<BM, BN, W, ST>::fits(a.D)) return hipErrorInvalidValue;
    if (out_mx) {
        if constexpr (BN % 32 == 0) {
            if (s16) hipLaunchKernelGGL((mid_mx_kernel<BM, BN, W, ST, 4, 1>), grid, block, 0, stream, a, tc);
            else hipLaunchKernelGGL((mid_mx_kernel<BM, BN, W, ST, 1, 1>), grid, block, 0, stream, a, tc);
        } else {
            return hipErrorInvalidValue;
        }
    } else {
        if (s16) hipLaunchKernelGGL((mid_mx_kernel<BM, BN, W, ST, 4, 0>), grid, block, 0, stream, a, tc);
        else hipLaunchKernelGGL((mid_mx_kernel<BM, BN, W, ST, 1, 0>), grid, block, 0, stream, a, tc);
    }
    return hipGetLastError();
}

struct MxMidShape {
    int bm, bn;
    bool (*fits)(int D);
};
const MxMidShape kMxMid[] = {
#define X(BM, BN, W, ST) {BM, BN, [](int D) { return MxMidCfg<BM, BN, W, ST>::fits(D); }},
    MXMID_CONFIGS(X)
#undef X
};
constexpr int kMxMidCount = sizeof(kMxMid) / sizeof(kMxMid[0]);

}  // namespace

// The small-tile configuration for R tokens, C weight rows and depth D, or -1
// where a tiled kernel takes less (tiled_us, its estimated time).  The price
// (us) is the bfloat16 one's (mid_plan) with the constants fitted to 2100
// measured times of these tiles over 208 sizes (1 to 1024 tokens): W from HBM
// at 6 TB/s, operands at 70 KB/us per CU, a launch with its scales 3, a
// further round 4.
int mx_mid_config(int R, int C, int D, int cus, int out_mx, double tiled_us) {
    if (R > 1024) return -1;
    const double depth = (double)((D + MXK - 1) / MXK) * MXK;
    const int cols = out_mx ? (C + 127) / 128 * 128 : C;
    const double hbm = 1e-6 * C * depth / 6.0;
    double best = tiled_us;
    int config = -1;
    for (int i = 0; i < kMxMidCount; ++i) {
        const int bm = kMxMid[i].bm, bn = kMxMid[i].bn;
        // the MX-FP8 output is written in whole 32-column blocks
        if ((out_mx && bn % 32) || (bm >= 32 && bm - 16 >= R) || !kMxMid[i].fits(D)) continue;
        const int64_t tiles = (int64_t)((R + bm - 1) / bm) * ((cols + bn - 1) / bn);
        const int64_t rounds = (tiles + cus - 1) / cus;
        const double load = rounds * (bm + bn) * depth / 70e3;
        const double t =
            3.0 + std::max(hbm, load) + 0.4 * std::min(hbm, load) + 4.0 * (rounds - 1) + 0.0006 * bm * bn;
        if (t < best) {
            best = t;
            config = i;
        }
    }
    return config;
}

hipError_t launch_mx_mid(const MxGemmArgs& a, int out_mx, int config, bool scales16, hipStream_t stream) {
    int i = 0;
#define X(BM, BN, W, ST) \
    if (config == i++) return launch_mx_mid_cfg<BM, BN, W, ST>(a, out_mx, scales16, stream);
    MXMID_CONFIGS(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace espace
