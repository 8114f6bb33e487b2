// 64 x 64 tiles on canonical codes for some hundred to about 1500 tokens: layers with one weight group, symmetric or asymmetric, whose K
// is whole chunks of 256 codes.
//
// With this few tiles a CU has one workgroup or two, and what counts is how often a wave stands and waits: the kernels of
// gemm_generic.hip and gemm_mid.hip walk K in steps of 128 codes with a barrier and a round trip through LDS each.  Here
//   * up to 1024 codes, all of K is in LDS at a time: every request is out before the first is waited for, and there is one barrier in
//     front of the products; longer K comes in chunks, the next of which is under way while one is multiplied;
//   * the requests go to LDS directly, rows as they lie with their 16-byte chunks swizzled; with K a constant their places are, too;
//   * eight waves: each takes a 32 x 32 quarter of the tile and half of K, or (long K: fewer reads from LDS and widenings per product, for
//     more sums to add up) 32 x 64 of it and a quarter of K; the operands of up to four blocks of 64 codes are read in one go;
//   * the integer sums of the shares meet in LDS, from where a thread takes eight channels of one row: 16-byte stores, and the
//     constants of the epilogue in registers since before the first request.
// us, before | here (K = 768: FN = 1, 3072: FN = 2, with the other form in brackets): 465 x 768 x 768 4.63 | 3.75 (3.88), asymmetric 4.86 |
// 4.06; 465 x 768 x 3072 7.25 | 6.39 (6.62), asymmetric 7.32 | 6.67 (6.71); 1024 x 1024 x 4096 9.5 | 8.05 (8.5); 1400 x 3072 x 768 asymmetric 14.7 |
// 11.8.  Three buffers of a chunk ahead instead of one change nothing at one workgroup to a CU and leave no room for a second:
// 465 x 768 x 3072 6.75, 1400 x 768 x 3072 9.8 -> 12.5.  Bound by the widening and, between barriers, by LDS: a chunk of 512 codes takes 0.6 us
// where its bytes take 0.3.
#include "gemm_common.hpp"

namespace w4a4 {
namespace {

typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr int kTile = 64;
constexpr int kSumPitch = 72;                                   // words from one row of sums to the next: four rows further is the other half of the banks
constexpr int tile_vmcnt(int n) { return (n & 0xF) | (0x7 << 4) | (0xF << 8) | (((n >> 4) & 0x3) << 14); }

// Position of 16-byte chunk c of row `row` inside the row, CPR chunks long: sixteen consecutive rows of one chunk start in sixteen
// different groups of four banks.
template <int CPR>
__device__ __forceinline__ int swizzle(int row) {
    static_assert(CPR % 8 == 0, "whole chunks of 256 codes");
    return CPR % 16 == 0 ? row & 15 : (row >> 1) & 7;
}

// NB x (1 + FN) operands of a wave, 16 bytes a lane.  The compiler does not see these reads (it would wait for every DMA in flight
// first, since it cannot tell which bytes a DMA writes); they are waited for in the same block.
template <int N>
__device__ __forceinline__ void lds_read(const uint32_t (&at)[N], v4f (&v)[N]) {
    static_assert(N == 3 || N == 4 || N == 6 || N == 8, "batches that are used");
    if constexpr (N == 3)
        asm volatile("ds_read_b128 %0, %3\nds_read_b128 %1, %4\nds_read_b128 %2, %5\ns_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]) : "v"(at[0]), "v"(at[1]), "v"(at[2]));
    if constexpr (N == 4)
        asm volatile("ds_read_b128 %0, %4\nds_read_b128 %1, %5\nds_read_b128 %2, %6\nds_read_b128 %3, %7\ns_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]) : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]));
    if constexpr (N == 6)
        asm volatile("ds_read_b128 %0, %6\nds_read_b128 %1, %7\nds_read_b128 %2, %8\nds_read_b128 %3, %9\nds_read_b128 %4, %10\nds_read_b128 %5, %11\n"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5])
                     : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]));
    if constexpr (N == 8)
        asm volatile("ds_read_b128 %0, %8\nds_read_b128 %1, %9\nds_read_b128 %2, %10\nds_read_b128 %3, %11\nds_read_b128 %4, %12\nds_read_b128 %5, %13\n"
                     "ds_read_b128 %6, %14\nds_read_b128 %7, %15\ns_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
                     : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]), "v"(at[7]));
}

// KCH: codes of K that are in LDS at a time, in NBUF buffers (1: all of K).  FN: column fragments of a wave.
template <int MODE, int OUT, int KCH, int NBUF, int FN>
__global__ __launch_bounds__(512) void gemm_tile64_kernel(GemmArgs g) {
    constexpr bool SGN = MODE == W4A4_SYM;
    constexpr int NW = 8, NT = NW * 64, KS = 2 * FN;            // waves; shares of K
    constexpr int CPR = KCH / 32;                               // 16-byte chunks of a row of KCH codes
    constexpr int OPB = kTile * CPR * 16, BUF = 2 * OPB;        // bytes of an operand, of a buffer
    constexpr int LD = CPR / NW;                                // DMA instructions per wave, operand and buffer
    static_assert(CPR % NW == 0, "every wave fetches as much");
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fi = wave & 1, fj = FN == 1 ? (wave >> 1) & 1 : 0, kw = FN == 1 ? wave >> 2 : wave >> 1;   // row half, first column half, share of K
    const int tile = xcd_tile(blockIdx.x, g.tiles_m * g.tiles_n);
    const int m0 = (tile / g.tiles_n) * kTile, n0 = (tile % g.tiles_n) * kTile;
    const int chunks = NBUF == 1 ? 1 : g.K / KCH;

    // ---- what the epilogue needs of this thread's row and eight channels, requested first of all ----------------------
    static_assert(kTile * 8 == NT, "a row's eight channels per thread");
    const int erow = tid >> 3, ecol = (tid & 7) * 8, n = n0 + ecol;
    const uint32_t noff = n < g.N ? (uint32_t)n : 0x10000000u;  // (N % 8 == 0: eight channels or none)
    const __amdgpu_buffer_rsrc_t sw_rsrc = make_rsrc(g.sw, (uint32_t)g.N * 4u);
    const __amdgpu_buffer_rsrc_t bias_rsrc = make_rsrc(g.bias, g.bias ? (uint32_t)g.N * 2u : 0u);
    const __amdgpu_buffer_rsrc_t zw_rsrc = make_rsrc(g.zw, SGN ? 0u : (uint32_t)g.N * 4u), c_rsrc = make_rsrc(g.c, SGN ? 0u : (uint32_t)g.N * 4u);
    u32x4 sw_raw[2], zw_raw[2], c_raw[2], bias_raw;
    float sa = 0.0f, za = 0.0f, ra = 0.0f;
    if constexpr (OUT != OUT_I32) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            sw_raw[k] = __builtin_amdgcn_raw_buffer_load_b128(sw_rsrc, noff * 4u + 16u * k, 0, 0);
            if constexpr (!SGN) {
                zw_raw[k] = __builtin_amdgcn_raw_buffer_load_b128(zw_rsrc, noff * 4u + 16u * k, 0, 0);
                c_raw[k] = __builtin_amdgcn_raw_buffer_load_b128(c_rsrc, noff * 4u + 16u * k, 0, 0);
            }
        }
        bias_raw = __builtin_amdgcn_raw_buffer_load_b128(bias_rsrc, noff * 2u, 0, 0);
        const int m = min(m0 + erow, g.M - 1);
        sa = g.sa[m];
        if constexpr (!SGN) { za = g.za[m]; ra = (float)g.RA[m]; }
    }

    // ---- global -> LDS: instruction i of this wave fills chunks 64 (i NW + wave) ..+63 of an operand ---------------------
    int voff_a[LD], voff_b[LD];
#pragma unroll
    for (int i = 0; i < LD; ++i) {
        const int q = (i * NW + wave) * 64 + lane, row = q / CPR, col = (q % CPR) ^ swizzle<CPR>(row);
        voff_a[i] = row * (int)g.lda + col * 16;
        voff_b[i] = row * (int)g.ldw + col * 16;
    }
    const int mrows = min(kTile, g.M - m0), nrows = min(kTile, g.N - n0);
    [[maybe_unused]] const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.Aq + (long)m0 * g.lda, (uint32_t)((long)(mrows - 1) * g.lda + g.K / 2));
    [[maybe_unused]] const __amdgpu_buffer_rsrc_t b_rsrc = make_rsrc(g.Wq + (long)n0 * g.ldw, (uint32_t)((long)nrows * g.ldw));
    auto fetch = [&](int c) {                                   // chunk c of K (past the last: turned away)
        uint8_t *dst = smem + (NBUF == 1 ? 0 : c % NBUF) * BUF + wave * 1024;
        const int gone = c < chunks ? 0 : (int)kPoison;
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the kernel's signature; it rejects the LDS cast
#pragma unroll
        for (int i = 0; i < LD; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, (lds_ptr_t)(dst + i * NW * 1024), 16, voff_a[i] | gone, c * (KCH / 2), 0, 0);
#pragma unroll
        for (int i = 0; i < LD; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, (lds_ptr_t)(dst + OPB + i * NW * 1024), 16, voff_b[i] | gone, c * (KCH / 2), 0, 0);
#else
        (void)dst; (void)gone;
#endif
    };
    constexpr int AHEAD = NBUF == 1 ? 1 : NBUF - 1;             // chunks requested before the first is waited for
#pragma unroll
    for (int c = 0; c < AHEAD; ++c) fetch(c);

    // ---- products ----------------------------------------------------------------------------------------------
    constexpr int KB = KCH / 64 / KS;                           // blocks of 64 codes per wave and chunk
    constexpr int NB = FN == 2 ? (KB % 2 ? 1 : 2) : KB % 4 == 0 ? 4 : KB % 3 == 0 ? 3 : KB % 2 == 0 ? 2 : 1;   // ... read at a time
    static_assert(KB >= 1 && KB % NB == 0, "whole batches");
    constexpr int NO = 1 + FN;                                  // operands of a block
    uint32_t base[NO], xr[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int row = o == 0 ? fi * 32 + r : (fj + o - 1) * 32 + r;
        base[o] = lds_address(smem) + (o ? OPB : 0) + row * CPR * 16;
        xr[o] = (uint32_t)(h ^ swizzle<CPR>(row)) << 4;
    }
    v16i acc[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[j][q] = 0;
    for (int c = 0; c < chunks; ++c) {
        __builtin_amdgcn_s_waitcnt(tile_vmcnt((AHEAD - 1) * 2 * LD));   // this wave's part of chunk c
        __builtin_amdgcn_s_barrier();                           // everyone's; and chunk c - 1 has been read
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        if constexpr (NBUF > 1) fetch(c + AHEAD);
        const uint32_t buf = NBUF == 1 ? 0u : (uint32_t)(c % NBUF) * BUF;
#pragma unroll
        for (int b0 = 0; b0 < KB; b0 += NB) {
            uint32_t at[NB * NO];
            v4f v[NB * NO];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int o = 0; o < NO; ++o) at[b * NO + o] = buf + base[o] + (xr[o] ^ (uint32_t)(kw * KB + b0 + b) * 32u);
            lds_read(at, v);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                v4i alo, ahi, lo[FN], hi[FN];
                widen<SGN>(__builtin_bit_cast(uint4, v[b * NO]), alo, ahi);
#pragma unroll
                for (int j = 0; j < FN; ++j) widen<SGN>(__builtin_bit_cast(uint4, v[b * NO + 1 + j]), lo[j], hi[j]);
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(alo, lo[j], acc[j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ahi, hi[j], acc[j], 0, 0, 0);
            }
        }
    }

    // ---- sums to rows: a copy per share of K, [64][kSumPitch]; then every thread takes eight channels of a row ---------------
    __builtin_amdgcn_s_waitcnt(tile_vmcnt(0));                  // no DMA may land in what follows
    __syncthreads();
    int *sums = reinterpret_cast<int *>(smem);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) sums[kw * (kTile * kSumPitch) + (fi * 32 + frag_row(0, q, lane)) * kSumPitch + (fj + j) * 32 + r] = acc[j][q];
    __syncthreads();
    constexpr int ESZ = OUT == OUT_F16 ? 2 : 4;
    const __amdgpu_buffer_rsrc_t o_rsrc = make_rsrc(g.out, (uint32_t)((long)g.M * g.N * ESZ));
    int P[8];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        v4i t = *reinterpret_cast<const v4i *>(sums + erow * kSumPitch + ecol + 4 * k);
#pragma unroll
        for (int o = 1; o < KS; ++o) t += *reinterpret_cast<const v4i *>(sums + (o * kTile + erow) * kSumPitch + ecol + 4 * k);
#pragma unroll
        for (int j = 0; j < 4; ++j) P[4 * k + j] = t[j];
    }
    const uint32_t off = n < g.N ? ((uint32_t)(m0 + erow) * (uint32_t)g.N + (uint32_t)n) * ESZ : kPoison;   // rows >= M fall off the end
    if constexpr (OUT == OUT_I32) {
        uint32_t o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = (uint32_t)(SGN ? P[j] >> 8 : P[j]);
        store_words<8>(o_rsrc, off, o);
    } else {
        // the operation order of tile_epilogue (one weight group), every operation rounded
        float y[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float sw = __uint_as_float(sw_raw[j >> 2][j & 3]);
            if constexpr (SGN) {
                const float t = (float)P[j] * sa;
                y[j] = t * (sw * 0.00390625f);
            } else {
                const float t1 = sw * (float)P[j], t2 = __uint_as_float(zw_raw[j >> 2][j & 3]) * ra;
                y[j] = sa * t1;
                const float u = sa * t2, z = za * __uint_as_float(c_raw[j >> 2][j & 3]);
                y[j] = y[j] + u;
                y[j] = y[j] + z;
            }
            const uint32_t b2 = bias_raw[j >> 1];
            if (g.bias) y[j] = y[j] + __half2float(__ushort_as_half((unsigned short)((j & 1) ? b2 >> 16 : b2 & 0xFFFFu)));
        }
        const bool gelu = g.act == W4A4_ACT_GELU;
        if constexpr (OUT == OUT_F32) {
            uint32_t o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] = __float_as_uint(gelu ? gelu_erf(y[j]) : y[j]);
            store_words<8>(o_rsrc, off, o);
        } else if (gelu) store_gelu_halves<8>(o_rsrc, off, y);
        else store_halves<8>(o_rsrc, off, y);
    }
}

template <int MODE, int OUT, int KCH, int NBUF, int FN>
int launch_tile(GemmArgs &g, hipStream_t st) {
    constexpr size_t codes = (size_t)NBUF * 2 * kTile * (KCH / 2), sums = (size_t)2 * FN * kTile * kSumPitch * 4, lds = codes > sums ? codes : sums;
    g.tiles_m = (g.M + kTile - 1) / kTile;
    g.tiles_n = (g.N + kTile - 1) / kTile;
    auto kern = gemm_tile64_kernel<MODE, OUT, KCH, NBUF, FN>;
    static KernelState ks;
    if (prepare_kernel(reinterpret_cast<const void *>(kern), lds, ks) < 0) return W4A4_ERR_HIP;
    const long tiles = (long)g.tiles_m * g.tiles_n;
    if (tiles > 0x7fffffffL) return W4A4_ERR_UNSUPPORTED_SHAPE;
    launch_gemm(kern, dim3((unsigned)tiles), dim3(512), lds, st, g);
    return launch_status();
}
// All of K at once up to 1024 codes, which leaves room for two workgroups on a CU; else two buffers of a chunk.
template <int MODE, int OUT>
int launch_k(GemmArgs &g, hipStream_t st) {
    switch (g.K) {
        case 256: return launch_tile<MODE, OUT, 256, 1, 1>(g, st);
        case 512: return launch_tile<MODE, OUT, 512, 1, 1>(g, st);
        case 768: return launch_tile<MODE, OUT, 768, 1, 1>(g, st);
        case 1024: return launch_tile<MODE, OUT, 1024, 1, 1>(g, st);
        default: return g.K % 512 == 0 ? launch_tile<MODE, OUT, 512, 2, 2>(g, st) : launch_tile<MODE, OUT, 256, 2, 2>(g, st);
    }
}
template <int MODE>
int launch_out(int out_kind, GemmArgs &g, hipStream_t st) {
    switch (out_kind) {
        case OUT_F16: return launch_k<MODE, OUT_F16>(g, st);
        case OUT_F32: return launch_k<MODE, OUT_F32>(g, st);
        case OUT_I32: return launch_k<MODE, OUT_I32>(g, st);
        default: return W4A4_ERR_INVALID_ARG;
    }
}

}  // namespace

// One weight group, K in chunks of 256 codes, rows within 32-bit offsets of a tile.  Asymmetric layers and long K always; symmetric ones of
// K < 1536 up to two tiles on each of 256 CUs (K = 256: one), beyond which the kernel of gemm_generic.hip, three and more
// workgroups of four waves to a CU, does without the sums in LDS (us, that kernel | this one: 600 x 3072 x 768, 480 tiles, 5.9 | 5.6, 1024 x 2304 x 768 (576)
// 6.9 | 6.8, 1400 x 3072 x 768 (1056) 9.6 | 10.1, 800 x 3072 x 1024 (624) 8.3 | 8.5; 1024 x 1024 x 256 (256) 3.47 | 3.41, 1400 x 1024 x 256
// (352) 3.9 | 4.2; 2000 x 1536 x 1536 (768) 11.3 | 10.8; asymmetric, against gemm_mid.hip, 1400 x 3072 x 768 14.7 | 11.8, 2000 x 1024 x 256 5.6 | 4.8).
// Chunks of 256 codes leave one such chunk ahead, where gemm_mid.hip has three steps ahead in each of four shares of K: K past 4096 in them goes there
// while there are too many tiles for one L2 to keep their operands and a CU for each (us, asymmetric, gemm_mid.hip | here, over rotating operands [over the same ones,
// which that L2 keeps]: 250 x 1600 x 4352 (100 tiles) 10.5 | 10.8 [8.6 | 8.0], x 5376 11.7 | 12.4 [9.6 | 9.0]; 1000 x 512 x 5376 (128) 11.2 | 12.4 [9.8 | 9.1]; 857 x 480 x 7936
// (112) 13.7 | 16.6 [12.3 | 11.8]; 506 x 240 x 6912 (32) 11.0 | 10.6; 780 x 1504 x 6400 (312) 18.1 | 16.1; in chunks of 512, 126 x 3832 x 4608 (120) 10.4 | 9.0).
bool tile64_ok(const GemmArgs &g, int mode) {
    if (g.ng != 1 || g.K % 256 || g.lda >= (1 << 24) || g.ldw >= (1 << 24)) return false;
    const long tiles = (long)((g.M + kTile - 1) / kTile) * ((g.N + kTile - 1) / kTile);
    if (g.K % 512 && g.K > 4096 && tiles > 32 && tiles <= 256) return false;
    return mode == W4A4_ASYM || g.K >= 1536 || tiles <= (g.K >= 512 ? 512 : 256);
}
int launch_tile64(int mode, int out_kind, GemmArgs &g, hipStream_t st) {
    return mode == W4A4_SYM ? launch_out<W4A4_SYM>(out_kind, g, st) : launch_out<W4A4_ASYM>(out_kind, g, st);
}

}  // namespace w4a4
