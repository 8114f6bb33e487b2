// Mid-sized problems (a few hundred to about 1500 tokens) on canonical codes: 64 x 64 tiles whose K range is
// split over KS pairs of waves.  Symmetric layers with one weight scale per output channel, and asymmetric
// layers with one weight group.
//
// With this few tiles a CU holds one workgroup or two, and a K step of 128 codes is a chain of latencies
// (fetch, barrier, LDS read, widening, dependent MFMAs: about 0.34 us on the 64 x 64 generic kernel), so the
// only cure is more of them at a time:
//   * wave pair p of the workgroup walks its own contiguous quarter (KS = 4) or half of K: 32 x 64 of the tile
//     per wave, int32 sums in registers, added up in LDS at the end (integers: any order gives the same sums);
//   * every pair has four LDS stages of its own, filled by 16-byte DMA three steps ahead: 96 KB in flight per
//     workgroup at KS = 4; unpadded rows with the XOR swizzle of gemm_olay.hip;
//   * the epilogue is dealt to all waves: a pair finishes 32 / KS rows of each of the tile's halves.
// What is left is the vector ALU of the widening (72 instructions per wave and step beside eight MFMAs): without the
// DMA a step takes 5 % less, without the MFMAs 20 %.  768 x 768 x 2176 8.2 -> 6.6 us against the generic kernel, asymmetric 12.9 -> 6.7; x 4224
// 18.6 -> 10.2 and 24.0 -> 10.4.  What is left to it is K in no whole chunks of 256 codes, and some long K (tile64_ok; the shares per shape: k_shares).
#include "gemm_common.hpp"

namespace w4a4 {
namespace {

typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int kMidTile = 64, kMidStage = 2 * kMidTile * (kBK / 2), kMidStages = 4;   // rows and columns; bytes per stage

constexpr int mid_vmcnt(int n) { return (n & 0xF) | (0x7 << 4) | (0xF << 8) | (((n >> 4) & 0x3) << 14); }

template <int MODE, int KS, int OUT>
__global__ __launch_bounds__(KS * 128) void gemm_mid_kernel(GemmArgs g) {
    constexpr bool SGN = MODE == W4A4_SYM;
    constexpr int QP = 4 / KS;                                  // four-row groups of a fragment that one wave finishes
    static_assert(KS == 2 || KS == 4, "a fragment's sixteen registers split into four-row groups");
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pair = wave >> 1, wm = wave & 1;                  // share of K; row half of the tile
    const int tile = xcd_tile(blockIdx.x, g.tiles_m * g.tiles_n);
    const int m0 = (tile / g.tiles_n) * kMidTile, n0 = (tile % g.tiles_n) * kMidTile;
    const int Kb = g.K / 2, KT = (g.K + kBK - 1) / kBK;
    const int steps = (KT + KS - 1) / KS, kt0 = pair * steps;   // (steps past K read zeros)

    // ---- DMA plan: instruction i of wave wm of a pair fills LDS rows 16 (2 i + wm) ..+15 of a stage (64 activation rows,
    // then 64 weight rows); lane l supplies physical slot l % 4 of row l / 4 = logical chunk (l % 4) ^ ((row >> 2) & 3)
    int voff[4], chunk[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (2 * i + wm) * 16 + (lane >> 2);
        chunk[i] = ((lane & 3) ^ ((row >> 2) & 3)) * 16;
        // LDS row p of the weight half holds channel 2 (p % 32) + p / 32: a lane ends up with two adjacent channels
        const int p = row - kMidTile;
        voff[i] = i < 2 ? row * (int)g.lda + chunk[i] : (2 * (p & 31) + (p >> 5)) * (int)g.ldw + chunk[i];
    }
    const int mrows = min(kMidTile, g.M - m0), nrows = min(kMidTile, g.N - n0);
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.Aq + (long)m0 * g.lda, (uint32_t)((long)(mrows - 1) * g.lda + Kb));
    const __amdgpu_buffer_rsrc_t b_rsrc = make_rsrc(g.Wq + (long)n0 * g.ldw, (uint32_t)((long)(nrows - 1) * g.ldw + Kb));
    uint8_t *ring = smem + pair * (kMidStages * kMidStage);
    auto fetch = [&](int s) {                                   // step s of this pair (past its range or K: zeros)
        const int kb = (kt0 + s) * (kBK / 2);
        const int left = s < steps ? Kb - kb : 0;
        uint8_t *dst = ring + (s & (kMidStages - 1)) * kMidStage + wm * 1024;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int vo = chunk[i] < left ? voff[i] : (int)kPoison;
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the kernel's signature; it rejects the LDS cast
            __builtin_amdgcn_raw_ptr_buffer_load_lds(i < 2 ? a_rsrc : b_rsrc, (lds_ptr_t)(dst + i * 2048), 16, vo, kb, 0, 0);
#else
            (void)vo; (void)dst;
#endif
        }
    };
    fetch(0);
    fetch(1);
    fetch(2);

    // ---- what the epilogue needs, requested before the main loop: this lane's two channels; the rows this wave finishes
    const int n_lane = n0 + 2 * (lane & 31);
    const bool n_ok = n_lane < g.N;                             // (N % 8 == 0: both channels or none)
    const int nc = n_ok ? n_lane : 0;
    float sw[2] = {0, 0}, bias[2] = {0, 0}, zw[2] = {0, 0}, cw[2] = {0, 0};
    float sa[QP][4], za[QP][4], ra[QP][4];
    if constexpr (OUT != OUT_I32) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            sw[j] = g.sw[nc + j] * (SGN ? 0.00390625f : 1.0f);
            if (g.bias) bias[j] = __half2float(g.bias[nc + j]);
            if (!SGN) { zw[j] = g.zw[nc + j]; cw[j] = g.c[nc + j]; }
        }
#pragma unroll
        for (int p = 0; p < QP; ++p)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int m = min(m0 + wm * 32 + 8 * (pair * QP + p) + 4 * (lane >> 5) + rr, g.M - 1);
                sa[p][rr] = g.sa[m];
                za[p][rr] = SGN ? 0.0f : g.za[m];
                ra[p][rr] = SGN ? 0.0f : (float)g.RA[m];
            }
    }

    // ---- main loop -------------------------------------------------------------------------------------------
    v16i acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0;
    const int swz = ((lane & 31) >> 2) & 3;
    const int rd = (lane & 31) * (kBK / 2) + (((lane >> 5) ^ swz) << 4);      // codes 0..63 of the step; 64..127: rd ^ 32
    for (int s = 0; s < steps; ++s) {
        __builtin_amdgcn_s_waitcnt(mid_vmcnt(8));               // this wave's part of step s has landed (two steps may be in flight)
        __builtin_amdgcn_s_barrier();                           // ... everyone's has, and step s - 1 has been read
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        fetch(s + 3);
        const uint32_t stage = lds_address(ring + (s & (kMidStages - 1)) * kMidStage);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint32_t off = stage + (uint32_t)(rd ^ (ks << 5));
            // (reads the compiler does not see: it would wait for every DMA in flight first)
            v4f a = lds_unseen_b128(off + wm * 2048), b0 = lds_unseen_b128(off + 4096), b1 = lds_unseen_b128(off + 6144);
            lds_unseen_wait(a); lds_unseen_also(b0); lds_unseen_also(b1);
            v4i alo, ahi, lo[2], hi[2];
            widen<SGN>(__builtin_bit_cast(uint4, a), alo, ahi);
            widen<SGN>(__builtin_bit_cast(uint4, b0), lo[0], hi[0]);
            widen<SGN>(__builtin_bit_cast(uint4, b1), lo[1], hi[1]);
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(alo, lo[j], acc[j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ahi, hi[j], acc[j], 0, 0, 0);
        }
    }

    // ---- add up the pairs' sums: red[pair][wm][j][r][lane]; a wave reads the four-row groups it finishes -----------
    __builtin_amdgcn_s_waitcnt(mid_vmcnt(0));                   // no DMA may land in what follows
    __syncthreads();
    int *red = reinterpret_cast<int *>(smem);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (q / QP != pair) {
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) red[((((pair * 2 + wm) * 2 + j) * 16) + 4 * q + rr) * 64 + lane] = acc[j][4 * q + rr];
            }
    __syncthreads();
    constexpr int ESZ = OUT == OUT_F16 ? 2 : 4;
    const __amdgpu_buffer_rsrc_t o_rsrc = make_rsrc(g.out, (uint32_t)((long)g.M * g.N * ESZ));
    const uint32_t row_bytes = (uint32_t)g.N * ESZ;
    const uint32_t col_off = n_ok ? (uint32_t)n_lane * ESZ : kPoison;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q / QP != pair) continue;                           // (uniform; keeps the register indices constants)
        const int p = q % QP;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            int P[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                P[j] = acc[j][4 * q + rr];
#pragma unroll
                for (int o = 1; o < KS; ++o)
                    P[j] += red[((((((pair + o) & (KS - 1)) * 2 + wm) * 2 + j) * 16) + 4 * q + rr) * 64 + lane];
            }
            const uint32_t off = (uint32_t)(m0 + wm * 32 + 8 * q + 4 * (lane >> 5) + rr) * row_bytes + col_off;
            if constexpr (OUT == OUT_I32) {
                const uint32_t w[2] = {(uint32_t)(SGN ? P[0] >> 8 : P[0]), (uint32_t)(SGN ? P[1] >> 8 : P[1])};
                store_words<2>(o_rsrc, off, w);
            } else {
                // the operation order of tile_epilogue (one weight group), every operation rounded
                float y[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if constexpr (SGN) {
                        const float t = (float)P[j] * sa[p][rr];
                        y[j] = t * sw[j];
                    } else {
                        const float t1 = sw[j] * (float)P[j], t2 = zw[j] * ra[p][rr];
                        y[j] = sa[p][rr] * t1;
                        const float u = sa[p][rr] * t2, z = za[p][rr] * cw[j];
                        y[j] = y[j] + u;
                        y[j] = y[j] + z;
                    }
                    if (g.bias) y[j] = y[j] + bias[j];
                }
                const bool gelu = g.act == W4A4_ACT_GELU;
                if constexpr (OUT == OUT_F32) {
                    const uint32_t w[2] = {__float_as_uint(gelu ? gelu_erf(y[0]) : y[0]), __float_as_uint(gelu ? gelu_erf(y[1]) : y[1])};
                    store_words<2>(o_rsrc, off, w);
                } else if (gelu) store_gelu_halves<2>(o_rsrc, off, y);
                else store_halves<2>(o_rsrc, off, y);
            }
        }
    }
}

template <int MODE, int KS, int OUT>
int launch_one(GemmArgs &g, hipStream_t st) {
    constexpr size_t lds = (size_t)KS * kMidStages * kMidStage;               // (the sums of the pairs need half of it)
    g.tiles_m = (g.M + kMidTile - 1) / kMidTile;
    g.tiles_n = (g.N + kMidTile - 1) / kMidTile;
    auto kern = gemm_mid_kernel<MODE, KS, OUT>;
    static KernelState ks;
    if (prepare_kernel(reinterpret_cast<const void *>(kern), lds, ks) < 0) return W4A4_ERR_HIP;
    const long tiles = (long)g.tiles_m * g.tiles_n;
    if (tiles > 0x7fffffffL) return W4A4_ERR_UNSUPPORTED_SHAPE;
    launch_gemm(kern, dim3((unsigned)tiles), dim3(KS * 128), lds, st, g);
    return launch_status();
}

template <int MODE, int KS>
int launch_out(int out_kind, GemmArgs &g, hipStream_t st) {
    switch (out_kind) {
        case OUT_F16: return launch_one<MODE, KS, OUT_F16>(g, st);
        case OUT_F32: return launch_one<MODE, KS, OUT_F32>(g, st);
        case OUT_I32: return launch_one<MODE, KS, OUT_I32>(g, st);
        default: return W4A4_ERR_INVALID_ARG;
    }
}

}  // namespace

// variant: the shares of K.  Requires one weight group, canonical codes, K % 32 == 0, lda % 16 == 0, operand matrices
// below 2^31 bytes.
int launch_mid(int variant, int mode, int out_kind, GemmArgs &g, hipStream_t st) {
    if (mode == W4A4_SYM) return variant == 2 ? launch_out<W4A4_SYM, 2>(out_kind, g, st) : launch_out<W4A4_SYM, 4>(out_kind, g, st);
    return variant == 2 ? launch_out<W4A4_ASYM, 2>(out_kind, g, st) : launch_out<W4A4_ASYM, 4>(out_kind, g, st);
}

}  // namespace w4a4
