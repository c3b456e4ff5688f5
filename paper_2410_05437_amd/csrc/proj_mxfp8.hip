// MX-FP8 projection (MX-FP8 output along the columns) of many tokens on tiles
// whose waves split the tile and every depth step.
//
// Eight waves, two per SIMD, as 2 x 2 over the tile and 2 over the depth: of
// every 128-deep step the waves of half h take codes 64 h .. 64 h + 63 for their
// quarter of the tile (v_mfma_scale_f32_32x32x64_f8f6f4; operand and result
// layouts in gemm_mxfp8.hip).  Three LDS stages; a wave reads the fragments of
// step t + 1 while it multiplies step t, so a step's stage is free one barrier
// after its fragments were read and receives step t + 3.  The halves' sums are
// added through LDS at the end, each wave finishing every other 32 x 32 block.
// Each XCD starts at another depth (MxDepthOrder).
//
// Four waves on the same tile, one per SIMD, took 1.0 us a step: a step's loads,
// its fragment reads (80 KB through LDS) and its 24 MFMAs a wave (0.37 us) came
// one after the other.  With two waves per SIMD and reads a step ahead they
// overlap: 0.85 us a step, 0.6 of it the 40 KB of operands through each CU's load
// path when nothing else runs.  No unit is saturated (4096 x 1536 x 4096: data return
// busy 58% of the time, L2 64%, MFMA 25%; the waves wait 42% of theirs).  Operands rotated through HBM, four
// waves -> this kernel: 4096 x 1536 x 4096 40 -> 35 us, x 11008 90 -> 82 (89 with
// all XCDs at the same depth), 2048 x 2458 x 6144 52 -> 47.  192 x 192 tiles (no
// registers left for reading ahead) and 256 x 128 ones in this scheme are slower
// or level with 128 x 128 tiles at every size tried.
#include "common.hpp"
#include "kernels.hpp"
#include "mx_core.hpp"

namespace espace {

namespace {

constexpr int PK = 128;                           // depth of a step: 128-byte rows

template <int BT, int BW, int SS>
struct PCfg {
    static constexpr int NS = 3;
    static constexpr int ROWS = BT + BW;
    static constexpr int DATA = ROWS * PK;
    // scale dwords: SS = 1, one per row after the codes of each stage; SS = 4
    // (scale rows 16-byte aligned), four steps' per row in two areas after the
    // stages, loaded with every fourth step
    static constexpr int STAGE = SS == 1 ? DATA + ROWS * 4 : DATA;
    static constexpr int SROW = 4 * SS;
    static constexpr int SAREA = ROWS * 16;
    static constexpr int NI = BT / 64, NJ = BW / 64;   // 32 x 32 blocks of a wave's quarter
    static constexpr int NB = NI * NJ;
    static constexpr int NDL = ROWS / 8;          // 1 KB code loads per stage
    static constexpr int LPD = (NDL + 7) / 8;     // per wave (uniform: extra ones repeat a load)
    static constexpr int NSL = ROWS / 64;         // scale loads (64 rows each), one per wave
    static constexpr int RING = NS * STAGE + (SS == 1 ? 0 : 2 * SAREA);
    static constexpr int RED = 8 * ((NB + 1) / 2) * 4096;
    static constexpr int SMEM = RING > RED ? RING : RED;
    static_assert(BT % 64 == 0 && BW % 64 == 0 && NSL <= 8 && SMEM <= 160 * 1024, "sizes");
    static_assert(SS == 1 || SS == 4, "scale steps");
    static __device__ __forceinline__ bool scales_with(int t) { return SS == 1 || (t & 3) == 0; }
};

template <int N>
__device__ __forceinline__ void p_wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// after this wave's LDS reads; its loads into LDS may stay in flight
__device__ __forceinline__ void p_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int NI, int NJ>
struct PFrag {
    i32x8_t t[NI], w[NJ];
    int ts[NI], ws[NJ];
};

// A lane's 32 code bytes of an LDS row: the 16-byte chunks at lo and hi.
__device__ __forceinline__ i32x8_t p_frag(const unsigned char* row, int lo, int hi) {
    const i32x4_t l = *reinterpret_cast<const i32x4_t*>(row + lo);
    const i32x4_t h = *reinterpret_cast<const i32x4_t*>(row + hi);
    return i32x8_t{l[0], l[1], l[2], l[3], h[0], h[1], h[2], h[3]};
}

template <int BT, int BW, int SS>
__global__ __launch_bounds__(512, 2)
void proj_mx_kernel(MxGemmArgs a, int tiles_c) {
    using C = PCfg<BT, BW, SS>;
    constexpr int NI = C::NI, NJ = C::NJ;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[C::SMEM];
    int tile_r, tile_c;
    tile_coords<8>(blockIdx.x, gridDim.x, tiles_c, 0, tile_r, tile_c);
    const int row0 = tile_r * BT, col0 = tile_c * BW;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = wave >> 2;                   // depth half of every step
    const int wt0 = ((wave >> 1) & 1) * (BT / 2), ww0 = (wave & 1) * (BW / 2);

    const auto tr = __builtin_amdgcn_make_buffer_rsrc((void*)a.T, (short)0, (int)(a.R * a.ldt), 0x00020000);
    const auto wr = __builtin_amdgcn_make_buffer_rsrc((void*)a.W, (short)0, (int)(a.C * a.ldw), 0x00020000);
    // load j of this wave covers rows 8 q .. 8 q + 7 of the tile (tokens
    // first), q = wave + 8 j; chunk c of row r sits at chunk c ^ ((r >> 1) & 7).
    // Rows past the matrix read its last row (their results are not stored).
    unsigned off[C::LPD];
#pragma unroll
    for (int j = 0; j < C::LPD; ++j) {
        const int q = min(wave + 8 * j, C::NDL - 1);
        const int rr = 8 * q + (lane >> 3);
        const int c = (lane & 7) ^ ((rr >> 1) & 7);
        off[j] = 16 * c + (unsigned)(8 * q < BT ? min(row0 + rr, a.R - 1) * (int)a.ldt
                                      : min(col0 + rr - BT, a.C - 1) * (int)a.ldw);
    }
    const int sl = wave % C::NSL;                 // this wave's scale load: rows 64 sl .. 64 sl + 63
    const bool stok = 64 * sl < BT;
    const int soff = stok ? min(row0 + 64 * sl + lane, a.R - 1) * (int)a.ldts
                          : min(col0 + 64 * sl + lane - BT, a.C - 1) * (int)a.ldws;
    const auto sr = __builtin_amdgcn_make_buffer_rsrc((void*)(stok ? a.Ts : a.Ws), (short)0,
                                                      (int)(stok ? a.R * a.ldts : a.C * a.ldws), 0x00020000);

    const int steps = (a.D + PK - 1) / PK;        // the codes are zero-padded to whole steps
    const MxDepthOrder order(steps);
    // the loads of step t into stage st; the 16-byte scale loads of a last
    // group may read past the matrix's steps (bytes never used; past the
    // buffer they read zeros)
    auto issue = [&](int t, int st) {
        unsigned char* stage = smem + st * C::STAGE;
        const int p = order(t);
#pragma unroll
        for (int j = 0; j < C::LPD; ++j) {
            const int q = min(wave + 8 * j, C::NDL - 1);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(8 * q < BT ? tr : wr,
                                                     (__attribute__((address_space(3))) void*)(stage + q * 1024), 16,
                                                     (int)off[j], p * PK, 0, 0);
        }
        if (C::scales_with(t)) {
            unsigned char* area = SS == 1 ? stage + C::DATA : smem + C::NS * C::STAGE + ((t >> 2) & 1) * C::SAREA;
            auto* dst = (__attribute__((address_space(3))) void*)(area + sl * 64 * C::SROW);
            if constexpr (SS == 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(sr, dst, 4, (int)soff, 4 * p, 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(sr, dst, 16, (int)soff, 4 * p, 0, 0);
        }
    };

    const int lr = lane & 31, lh = lane >> 5;
    const int sw = (lr >> 1) & 7;
    const int c_lo = ((4 * half + lh) ^ sw) << 4, c_hi = ((4 * half + 2 + lh) ^ sw) << 4;
    const int t_row = wt0 + lr, w_row = BT + ww0 + lr;
    using Frag = PFrag<NI, NJ>;
    auto read = [&](Frag& f, int t, int st) {
        const unsigned char* stage = smem + st * C::STAGE;
        const unsigned char* sc = (SS == 1 ? stage + C::DATA
                                           : smem + C::NS * C::STAGE + ((t >> 2) & 1) * C::SAREA + 4 * (t & 3)) +
                                  2 * half + lh;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            f.t[i] = p_frag(stage + (t_row + 32 * i) * PK, c_lo, c_hi);
            f.ts[i] = sc[4 * SS * (t_row + 32 * i)];
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            f.w[j] = p_frag(stage + (w_row + 32 * j) * PK, c_lo, c_hi);
            f.ws[j] = sc[4 * SS * (w_row + 32 * j)];
        }
    };

    f32x16_t acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    Frag f0, f1;
    for (int t = 0; t < 3 && t < steps; ++t) issue(t, t);
    p_wait_vm<0>();
    p_barrier();
    read(f0, 0, 0);
    int st = 0;                                   // stage of step t
    auto step = [&](const Frag& cur, Frag& nxt, int t) {
        // this wave's loads of step t + 1 have landed (those of step t + 2 may
        // stay in flight); after the barrier every wave's have, and every wave
        // has its fragments of step t: its stage receives step t + 3 (a scale
        // area is rewritten only when the four steps after its own are loaded
        // and its last step's scales were read)
        if (t + 2 < steps) {
            if (C::scales_with(t + 2)) p_wait_vm<C::LPD + 1>();
            else p_wait_vm<C::LPD>();
        } else {
            p_wait_vm<0>();
        }
        p_barrier();
        if (t + 3 < steps) issue(t + 3, st);
        st = st == 2 ? 0 : st + 1;
        read(nxt, t + 1, st);                     // after the last step: of no use, inside the ring
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cur.w[j], cur.t[i], acc[i][j], 0, 0, 0,
                                                                            cur.ws[j], 0, cur.ts[i]);
        __builtin_amdgcn_sched_barrier(0);
    };
    int t = 0;
    for (; t + 1 < steps; t += 2) {
        step(f0, f1, t);
        step(f1, f0, t + 1);
    }
    if (t < steps) step(f0, f1, t);

    // ---- the halves' sums: a wave gives the blocks of the other parity to the
    // wave of the other half and finishes those of its own half's parity.  The
    // last step waited for every load into LDS.
    __syncthreads();
    f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);
    constexpr int PER = (C::NB + 1) / 2;
#pragma unroll
    for (int b = 0; b < C::NB; ++b) {
        if ((b & 1) == half) continue;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x16_t& v = acc[b / NJ][b % NJ];
            red[((wave * PER + b / 2) * 4 + g) * 64 + lane] = f32x4_t{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        }
    }
    __syncthreads();
    // register r of block (i, j) holds token row wt0 + 32 i + lr and output
    // column ww0 + 32 j + 8 (r / 4) + 4 lh + r % 4: a block is one 32-column
    // MX block of 32 tokens, each in lanes l and l + 32
    uint8_t* Zq = static_cast<uint8_t*>(a.out);
#pragma unroll
    for (int b = 0; b < C::NB; ++b) {
        if ((b & 1) != half) continue;
        const int n = row0 + wt0 + 32 * (b / NJ) + lr;
        const int cb = col0 + ww0 + 32 * (b % NJ);
        float v[16];
        float amax = 0.f;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4_t o = red[(((wave ^ 4) * PER + b / 2) * 4 + g) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float s = acc[b / NJ][b % NJ][4 * g + e] + o[e];
                v[4 * g + e] = cb + 8 * g + 4 * lh + e < a.C ? s : 0.f;
                amax = fmaxf(amax, fabsf(v[4 * g + e]));
            }
        }
        amax = fmaxf(amax, __shfl_xor(amax, 32));
        const int sb = mx_scale_byte(amax);
        const int nsh = 127 - sb;                 // multiply by 2^-S
        uint32_t w[4];
#pragma unroll
        for (int g = 0; g < 4; ++g)
            w[g] = mx_pack4(__builtin_amdgcn_ldexpf(v[4 * g], nsh), __builtin_amdgcn_ldexpf(v[4 * g + 1], nsh),
                            __builtin_amdgcn_ldexpf(v[4 * g + 2], nsh), __builtin_amdgcn_ldexpf(v[4 * g + 3], nsh));
        // after the swaps with the lane 32 away, lane half lh holds the 16
        // codes of columns cb + 16 lh .. + 15
        const auto p02 = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto p13 = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        if (n < a.R && cb < a.cpad) {
            const int c = cb + 16 * lh;
            // row pairs: columns cb .. cb + 31 lie in one 64-code block
            uint8_t* p = Zq + (a.out_pairs ? (int64_t)(n >> 1) * a.ldo + (c >> 6) * 128 + (n & 1) * 64 + (c & 63)
                                           : (int64_t)n * a.ldo + c);
            *reinterpret_cast<u32x4_t*>(p) = u32x4_t{p02[0], p02[1], p13[0], p13[1]};
            if (lh == 0) a.outs[(int64_t)n * a.ldos + cb / 32] = (uint8_t)sb;
        }
    }
}

template <int BT, int BW>
hipError_t launch_cfg(const MxGemmArgs& a, bool scales16, hipStream_t stream) {
    const int tiles_c = (a.cpad + BW - 1) / BW;   // the padding columns are written too
    const int tiles = tiles_c * ((a.R + BT - 1) / BT);
    if (scales16)
        hipLaunchKernelGGL((proj_mx_kernel<BT, BW, 4>), dim3(tiles), dim3(512), 0, stream, a, tiles_c);
    else
        hipLaunchKernelGGL((proj_mx_kernel<BT, BW, 1>), dim3(tiles), dim3(512), 0, stream, a, tiles_c);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_proj_mx(const MxGemmArgs& a, bool scales16, hipStream_t stream) {
    return launch_cfg<128, 192>(a, scales16, stream);
}

}  // namespace espace
