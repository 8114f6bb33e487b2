// Linear layer for small token counts with the activation quantize inside the GEMM kernel:
//   out = epilogue( Q(X) * Wq^T ),  Q = the symmetric per-token INT4 mapping of Sec. 3.1.
//
// At batch 1 x sequence 128 (M = 128) a linear layer is a few microseconds of work and the
// launch of a kernel costs about as much (Sec. 4.2: at small batch x sequence the launch overhead
// and the memory-bound quantize kernels are what hurts).  So this path spends arithmetic to save
// a launch: every workgroup quantizes the rows of its 32 tokens itself, into LDS, and multiplies
// from there; codes and scales never reach memory.  The result is bit for bit what
// w4a4_quantize_act followed by w4a4_linear gives (same fp32 operations in the same order, exact
// integer sums).
//
//   * tile: 32 tokens x 32 (or 64) channels per workgroup of NW = 4, 8 or 16 waves;
//   * pass 1: the 32 x K fp16 rows are read ONCE, fully coalesced (2 NW consecutive lanes per token),
//     and stay in registers (at most 16 chunks of 16 bytes per lane) while the range of each token
//     is reduced over its lanes; then every lane quantizes its own registers: t = x * (7/absmax),
//     rne(t) by adding 1.5 * 2^23 (the clamp of the mapping cannot bind for symmetric codes); the
//     code then sits in the low byte of the sum and v_perm_b32 gathers four of them into an int8
//     MFMA operand register, in the order the weight widening produces (even codes, odd codes of
//     a packed dword).  The int8 tile goes to LDS (row pitch K + 16 bytes: conflict-free 16-byte
//     reads of 32 consecutive rows);
//   * the packed weight codes of the tile's channels are requested together with the activation
//     rows, coalesced as well, and parked in LDS beside the activation codes;
//   * pass 2: the waves split K in blocks of 64 codes (interleaved) and read both operands from
//     LDS in MFMA order; weights are widened to 16 * code, activations stay 1 * code: the
//     accumulators hold 16 * P;
//   * the int32 partial sums of the waves are added in LDS and the accumulator registers of the
//     tile are dealt round robin to the waves for the epilogue.
#include "gemm_common.hpp"
#include "layer.hpp"

namespace w4a4 {

struct SmallArgs {
    const __half *X; long ldx;       // [M, K] fp16, row stride in elements (fp16-activation form)
    const uint8_t *Aq; long lda;     // [M, K/2] canonical packed codes, row stride in bytes (packed form)
    const float *sa;                 // [M] token scales (packed form)
    const float *za; const int32_t *RA;   // [M] zero points, code sums (packed unsigned codes)
    const float *zw, *c;             // [N] weight zero points, row sums (packed unsigned codes)
    int32_t *acc_out;                // packed form only: store the int32 sums P [M, N] instead of fp16 outputs
    const uint8_t *Wq; long ldw;     // canonical packed codes [N, K/2]; INT8 sibling: int8 codes [N, K]
    const float *sw;                 // [N]
    const __half *bias; int act;
    __half *out;                     // [M, N]
    int M, N, K, tiles_n;
    uint32_t wcpr_inv;               // 2^32 / (16-byte chunks of a row of weights), rounded up: p * wcpr_inv >> 32 is the row of chunk p < 2^16
    // LayerNorm form: the activations are LN(X + R) gamma + beta in fp16, which also go to Y
    const __half *R, *gamma, *beta;  // [M, K] dense, [K], [K]
    float eps;
    __half *Y;                       // [M, K]
};

// 16-byte chunks held by one lane: of its token row (K <= 4096: 512 chunks over 2 NW * 32 / TM lanes), and of
// the weight tile on its way to LDS (the launcher checks the latter)
constexpr int small_xchunks(int tm) { return tm == 16 ? 8 : 16; }
constexpr int small_wchunks(int nw) { return nw == 16 ? 4 : 6; }

// eight fp16 values -> their codes, as two operand registers: bytes (c0,c2,c4,c6) and (c1,c3,c5,c7)
// (NATURAL: bytes (c0,c1,c2,c3) and (c4,c5,c6,c7) instead: the order of one-byte weight codes)
template <bool NATURAL = false>
__device__ __forceinline__ void codes8(const u32x4 &x, float inv, uint32_t &even, uint32_t &odd) {
    uint32_t u[8];
    const float nzero = -0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // t = fp32(x) * inv in one instruction: v_fma_mix_f32 reads the fp16 half directly and rounds the
        // product once to fp32 (the addend -0 changes nothing), exactly what convert-then-multiply gives
        float t0, t1;
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(t0) : "v"(x[i]), "v"(inv), "v"(nzero));
        asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(t1) : "v"(x[i]), "v"(inv), "v"(nzero));
        u[2 * i] = __float_as_uint(t0 + 12582912.0f);
        u[2 * i + 1] = __float_as_uint(t1 + 12582912.0f);
    }
    if (NATURAL) {
        even = __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0400u) | __builtin_amdgcn_perm(u[3], u[2], 0x04000c0cu);
        odd = __builtin_amdgcn_perm(u[5], u[4], 0x0c0c0400u) | __builtin_amdgcn_perm(u[7], u[6], 0x04000c0cu);
    } else {
        even = __builtin_amdgcn_perm(u[2], u[0], 0x0c0c0400u) | __builtin_amdgcn_perm(u[6], u[4], 0x04000c0cu);
        odd = __builtin_amdgcn_perm(u[3], u[1], 0x0c0c0400u) | __builtin_amdgcn_perm(u[7], u[5], 0x04000c0cu);
    }
}

// The LayerNorm form.  X + R, normalised, scaled and shifted: bit for bit what layernorm_quantize_kernel makes of a row of K = 512,
// 768 or 1024, whose thirty-two lanes hold chunks l + 32 it.  Here LPR = 32 lanes hold the same chunks, or sixteen hold
// l + 16 i, of which the even i are lane l's there and the odd i lane l + 16's: the sums are formed apart and joined last.
// Every operation is rounded as there; v_fma_mix_f32 takes its fp16 operands without converting them first (with a factor
// of 1 or an addend of -0, which leave one rounding).  On return x holds the row's fp16 values.
__device__ __forceinline__ float mix_add(uint32_t a, uint32_t b, int hi) {          // fp16 half of a + fp16 half of b
    float d;
    if (hi) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(a), "v"(b));
    else asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
__device__ __forceinline__ float mix_mul(float y, uint32_t g, int hi) {             // y * fp16 half of g
    float d;
    const float nzero = -0.0f;
    if (hi) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,1,0] op_sel_hi:[0,1,0]" : "=v"(d) : "v"(y), "v"(g), "v"(nzero));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,0,0] op_sel_hi:[0,1,0]" : "=v"(d) : "v"(y), "v"(g), "v"(nzero));
    return d;
}
__device__ __forceinline__ float mix_add_half(float y, uint32_t b, int hi) {        // y + fp16 half of b
    float d;
    if (hi) asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(d) : "v"(y), "v"(b));
    else asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[0,0,1]" : "=v"(d) : "v"(y), "v"(b));
    return d;
}
template <int LPR>
__device__ __forceinline__ float row_total(float s0, float s1) {
    auto add = [](float p, float q) { return p + q; };
    if constexpr (LPR == 32) return lanes_reduce<32>(s0, add);
    return lanes_reduce<16>(s0, add) + lanes_reduce<16>(s1, add);
}
template <int LPR, int XCH, int K>
__device__ __forceinline__ void layernorm_row(u32x4 (&x)[XCH], const u32x4 (&r)[XCH], const u32x4 (&g)[XCH], const u32x4 (&b)[XCH], float eps) {
    static_assert((LPR == 16 || LPR == 32) && XCH * LPR * 8 == K, "lanes of a row");
    float v[XCH][8];
    constexpr float inv_k = 1.0f / (float)K;
    float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
    for (int i = 0; i < XCH; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[i][e] = mix_add(x[i][e / 2], r[i][e / 2], e & 1);
            if (LPR == 32 || i % 2 == 0) s0 += v[i][e];
            else s1 += v[i][e];
        }
    const float mean = row_total<LPR>(s0, s1) * inv_k;
    s0 = s1 = 0.0f;
#pragma unroll
    for (int i = 0; i < XCH; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[i][e] = v[i][e] - mean;
            const float d2 = v[i][e] * v[i][e];
            if (LPR == 32 || i % 2 == 0) s0 += d2;
            else s1 += d2;
        }
    const float var = row_total<LPR>(s0, s1) * inv_k;
    const float rstd = 1.0f / sqrtf(var + eps);
#pragma unroll
    for (int i = 0; i < XCH; ++i)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            float y[2];
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) y[hi] = mix_add_half(mix_mul(v[i][2 * p + hi] * rstd, g[i][p], hi), b[i][p], hi);
            const __half2 h = __floats2half2_rn(y[0], y[1]);
            x[i][p] = *reinterpret_cast<const uint32_t *>(&h);
        }
}

// NW waves, FN column fragments of 32 channels, TM = 32, 16 or 8 tokens per workgroup (with fewer than 32 the upper
// MFMA rows repeat the lower ones and are not stored), WLDS: the weight tile is staged in LDS.
// PACKED: the activations arrive already quantized (packed codes + token scales, the output of
// w4a4_quantize_act or of a producer kernel): pass 1 only parks their tile in LDS, and both operands are
// widened to 16 * code on their way into the MFMA (the sums hold 256 * P).
// W8: the INT8 sibling.  Tokens are quantized with 127 levels per side (or arrive as one int8 code per
// byte when PACKED), the weights are one int8 code per byte, and both go into the MFMA as they are (the
// sums hold P).
// ASYM (packed codes only): unsigned codes, one weight group; the sums hold P and the epilogue adds the zero-point terms.
// KC: 0, or K.  What bounds these kernels is the instructions a wave issues one behind the other (a dependent one every 8 cycles; a launch
// by itself takes 1.5 us of such a stream, a request answered from L2 0.1), and a third of them worked out addresses: with K a
// constant, offsets, trip counts and places in LDS are, too.  Back to back, us, before | K a run-time value, tile rows by a product instead of a
// division and carries | K a constant, which also unrolls pass 2: fp16 activations 32 x 2304 x 768 4.31 | - | 2.95, 128 x 2304 x 768 6.04 | - | 4.17,
// 32 x 768 x 3072 6.14 | - | 4.08; packed 32 x 2304 x 768 3.37 | 3.24 | 2.44, 128 x 768 x 3072 4.18 | 4.14 | 3.50.  One layer of 768 features, 1 x 32
// tokens, 26.6 -> 22.2, 1 x 128 31.7 -> 26.3.
// LN (with KC): the activations are the LayerNorm of X + R, which every workgroup forms for its tokens; the first column tile
// stores them.
template <int NW, int FN, int TM, bool WLDS, bool PACKED, bool W8 = false, bool ASYM = false, int KC = 0, bool LN = false>
__global__ __launch_bounds__(NW * 64) void linear_f16act_kernel(SmallArgs a) {
    constexpr int NT = NW * 64, LPR = NT / TM;                  // LPR consecutive lanes share a token in pass 1
    constexpr int RV = TM / 2;                                  // accumulator registers per fragment that hold real rows
    constexpr int R = RV * FN;                                  // ... of the tile
    constexpr int RPW = (RV + NW - 1) / NW;                     // rows' registers finished by one wave, for all column fragments
    // Column fragments: a wave takes one of them and a larger share of K (half of the sums to add up in LDS: 128 x 2304 x 768 4.5 us ->
    // 4.2), or all of them where K is no constant or the weights come from memory, which shares the other operand.
    constexpr int FPW = KC && WLDS ? 1 : FN, KW = NW * FPW / FN;   // fragments of a wave, waves that share out K
    const int K = KC ? KC : a.K;
    constexpr int WCH = !WLDS ? 1 : KC ? (32 * FN * (W8 ? KC / 16 : KC / 32) + NT - 1) / NT : small_wchunks(NW);
    constexpr int XCH = PACKED ? 1 : KC ? KC / 8 / LPR : small_xchunks(TM);
    static_assert(!LN || (KC && !PACKED && !W8 && NW == 8), "fp16 activations of up to 1024 features");
    static_assert(KC == 0 || PACKED || KC % (8 * LPR) == 0, "whole chunks for each lane of a row");
    constexpr int ACH = !PACKED ? 1 : KC ? (TM * (W8 ? KC / 16 : KC / 32) + NT - 1) / NT : W8 ? 8 : 4;   // 16-byte chunks of the packed activation tile per lane
    constexpr bool NIBBLES = PACKED && !W8;                     // activation codes arrive two per byte
    static_assert(!ASYM || NIBBLES, "unsigned codes arrive packed");
    static_assert(LPR <= 64 && (LPR & (LPR - 1)) == 0, "a token's lanes sit in one wave");
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int wpitch = (W8 ? K : K / 2) + 16, pitch = NIBBLES ? K / 2 + 16 : K + 16;
    uint8_t *codes = smem;                                      // [TM][pitch] int8 activation codes (packed codes if PACKED)
    uint8_t *wt = codes + TM * pitch;                           // [32 FN][wpitch] packed weight codes (WLDS)
    int *s_sum = reinterpret_cast<int *>(wt + (WLDS ? 32 * FN * wpitch : 0));   // [R][64]
    float *s_S = reinterpret_cast<float *>(s_sum + R * 64);     // [TM] (ASYM: scales, zero points, code sums)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = (blockIdx.x / a.tiles_n) * TM, n0 = (blockIdx.x % a.tiles_n) * (32 * FN);
    const __amdgpu_buffer_rsrc_t x_rsrc = PACKED ? make_rsrc(a.Aq, (uint32_t)((long)(a.M - 1) * a.lda + (W8 ? K : K / 2)))
                                                 : make_rsrc(a.X, (uint32_t)(((long)(a.M - 1) * a.ldx + K) * 2));
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(a.Wq, (uint32_t)((long)a.N * a.ldw));
    const int r = lane & 31, h = lane >> 5;                     // pass 2: token / channel r, K half h
    const int nb = K / 64;

    // ---- requests, in the order they are needed: activation rows, weights, channel constants ----------------
    const int row = tid / LPR, c0 = tid % LPR;
    const int nchunks = K / 8;                                  // 16-byte chunks of an activation row
    const int wcpr = W8 ? K / 16 : K / 32;                      // 16-byte chunks of a row of weight codes
    u32x4 x[XCH];
    [[maybe_unused]] u32x4 rx[LN ? XCH : 1], gx[LN ? XCH : 1], bx[LN ? XCH : 1];
    u32x4 ast[ACH];
    auto row_of = [&](int p) { return KC ? p / wcpr : (int)__umulhi((uint32_t)p, a.wcpr_inv); };   // row of chunk p of a tile of codes
    if constexpr (!PACKED) {
        const uint32_t base = (uint32_t)min(m0 + row, a.M - 1) * (uint32_t)a.ldx * 2u;
#pragma unroll
        for (int i = 0; i < XCH; ++i)               // (chunks past the row are requested but never used)
            if (i * LPR < nchunks) x[i] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, base + (uint32_t)(c0 + i * LPR) * 16, 0, 0);
        if constexpr (LN) {
            const __amdgpu_buffer_rsrc_t r_rsrc = make_rsrc(a.R, (uint32_t)((long)a.M * K * 2));
            const __amdgpu_buffer_rsrc_t g_rsrc = make_rsrc(a.gamma, (uint32_t)K * 2u), be_rsrc = make_rsrc(a.beta, (uint32_t)K * 2u);
            const uint32_t rbase = (uint32_t)min(m0 + row, a.M - 1) * (uint32_t)K * 2u;
#pragma unroll
            for (int i = 0; i < XCH; ++i)
                if (i * LPR < nchunks) rx[i] = __builtin_amdgcn_raw_buffer_load_b128(r_rsrc, rbase + (uint32_t)(c0 + i * LPR) * 16, 0, 0);
#pragma unroll
            for (int i = 0; i < XCH; ++i)
                if (i * LPR < nchunks) {
                    gx[i] = __builtin_amdgcn_raw_buffer_load_b128(g_rsrc, (uint32_t)(c0 + i * LPR) * 16, 0, 0);
                    bx[i] = __builtin_amdgcn_raw_buffer_load_b128(be_rsrc, (uint32_t)(c0 + i * LPR) * 16, 0, 0);
                }
        }
    } else {
        // the packed tile (rows past M fall outside the descriptor: zeros): chunk p is chunk p % wcpr of row p / wcpr
#pragma unroll
        for (int i = 0; i < ACH; ++i) {                         // (chunks past the tile: turned away, cheaper than a branch around each)
            const int p = tid + i * NT, rw = row_of(p);
            const uint32_t off = (uint32_t)(m0 + rw) * (uint32_t)a.lda + (uint32_t)(p - rw * wcpr) * 16;
            ast[i] = __builtin_amdgcn_raw_buffer_load_b128(x_rsrc, p < TM * wcpr ? off : kPoison, 0, 0);
        }
    }
    // (packed form) constants of the tile's tokens, for wave 0 to pass on; in front of the weights, which nobody has to wait for here
    float sa_m = 0.0f, za_m = 0.0f;
    int ra_m = 0;
    if (PACKED && wave == 0) {
        const int m = min(m0 + lane % TM, a.M - 1);
        sa_m = a.sa[m];
        if constexpr (ASYM) { za_m = a.za[m]; ra_m = a.RA[m]; }
    }
    // weights: the whole tile, on its way to LDS; when it does not fit there, pass 2 fetches its operands itself (lane (c, h): 16
    // bytes of channel c).  Rows of weights are dense, so the tile is one piece of memory and chunk p of it 16 p bytes from its start:
    // which row that is matters only for the place in LDS, worked out while the requests are under way.
    u32x4 wst[WCH];
    if constexpr (WLDS) {
        const uint32_t src = (uint32_t)n0 * (uint32_t)a.ldw + (uint32_t)tid * 16;
#pragma unroll
        for (int i = 0; i < WCH; ++i)
            wst[i] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, tid + i * NT < 32 * FN * wcpr ? src + (uint32_t)(i * NT) * 16 : kPoison, 0, 0);
    }
    // pass 2: wave kw of the KW that share out K for column fragments j0 ..  Lane r of fragment j holds channel FN r + j of the tile, so
    // that a lane ends up with FN adjacent channels; with weights from memory 32 j + r, since the rows that a request reads
    // had better be neighbours (every second row of 2 KB: 300 x 1024 x 4096 7.4 us -> 8.7)
    constexpr bool ADJ = WLDS || FN == 1;
    auto channel = [&](int j) { return n0 + (ADJ ? FN * r + j : 32 * j + r); };
    const int j0 = FPW == FN ? 0 : wave % FN, kw = wave * FPW / FN;
    constexpr int NBW = KC ? (KC / 64 + KW - 1) / KW : 1;       // blocks of 64 codes per wave
    // Weights from memory: all of them requested here, where quantizing the tokens takes its time (300 x 1024 x 4096 11.2 us -> 10.7);
    // behind packed activations they would only stand in each other's way (7.0 us -> 8.4)
    constexpr bool WPRE = !WLDS && KC && !W8 && !PACKED;
    u32x4 wpre[WPRE ? NBW : 1][FPW];
    auto request_w = [&](int j, int b) {
        return __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, (uint32_t)channel(j) * (uint32_t)a.ldw + (uint32_t)(b * 32 + h * 16), 0, 0);
    };
    if constexpr (WPRE) {
#pragma unroll
        for (int i = 0; i < NBW; ++i)
            if (kw + i * KW < nb) {
#pragma unroll
                for (int j = 0; j < FPW; ++j) wpre[i][j] = request_w(j0 + j, kw + i * KW);
            }
    }
    // constants of this lane's channels, as raw bits: nothing here waits for a load
    const __amdgpu_buffer_rsrc_t sw_rsrc = make_rsrc(a.sw, (uint32_t)a.N * 4u);
    const __amdgpu_buffer_rsrc_t b_rsrc = make_rsrc(a.bias, a.bias ? (uint32_t)a.N * 2u : 0u);   // no bias: reads zero
    const __amdgpu_buffer_rsrc_t zw_rsrc = make_rsrc(a.zw, ASYM ? (uint32_t)a.N * 4u : 0u);
    const __amdgpu_buffer_rsrc_t c_rsrc = make_rsrc(a.c, ASYM ? (uint32_t)a.N * 4u : 0u);
    uint32_t sw_raw[FN], zw_raw[ASYM ? FN : 1], c_raw[ASYM ? FN : 1];
    unsigned short b_raw[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        sw_raw[j] = __builtin_amdgcn_raw_buffer_load_b32(sw_rsrc, (uint32_t)channel(j) * 4u, 0, 0);
        b_raw[j] = __builtin_amdgcn_raw_buffer_load_b16(b_rsrc, (uint32_t)channel(j) * 2u, 0, 0);
        if constexpr (ASYM) {
            zw_raw[j] = __builtin_amdgcn_raw_buffer_load_b32(zw_rsrc, (uint32_t)channel(j) * 4u, 0, 0);
            c_raw[j] = __builtin_amdgcn_raw_buffer_load_b32(c_rsrc, (uint32_t)channel(j) * 4u, 0, 0);
        }
    }
    for (int e = tid; e < R * 64; e += NT) s_sum[e] = 0;

    // ---- pass 1: ranges, codes into LDS ----------------------------------------------------------------------
    if constexpr (PACKED) {
#pragma unroll
        for (int i = 0; i < ACH; ++i) {
            const int p = tid + i * NT;
            if (p < TM * wcpr) *reinterpret_cast<u32x4 *>(codes + (p + row_of(p)) * 16) = ast[i];
        }
        if (tid < TM) {
            s_S[tid] = sa_m;
            if constexpr (ASYM) { s_S[TM + tid] = za_m; s_S[2 * TM + tid] = (float)ra_m; }
        }
    } else {
        if constexpr (LN) {
            layernorm_row<LPR, XCH, KC>(x, rx, gx, bx, a.eps);
            if (n0 == 0 && m0 + row < a.M) {
#pragma unroll
                for (int i = 0; i < XCH; ++i)
                    if (i * LPR < nchunks) *reinterpret_cast<u32x4 *>(a.Y + (long)(m0 + row) * K + (c0 + i * LPR) * 8) = x[i];
            }
        }
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        uint32_t zero = 0;
        h2 mx = *reinterpret_cast<const h2 *>(&zero);
#pragma unroll
        for (int i = 0; i < XCH; ++i) {
            if (i * LPR < nchunks && c0 + i * LPR < nchunks) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t d = x[i][k] & 0x7FFF7FFFu;
                    mx = __builtin_elementwise_max(mx, *reinterpret_cast<const h2 *>(&d));
                }
            }
        }
        float amax = fmaxf((float)mx[0], (float)mx[1]);
        amax = lanes_reduce<LPR>(amax, [](float p, float q) { return fmaxf(p, q); });
        Range rg = range_sym(amax);
        if (W8) {                                                // Sec. 3.1 with b = 8: 127 levels per side
            if (amax == 0.0f) { rg.inv = 0.0f; rg.S = 1.0f; }
            else { rg.inv = 127.0f / amax; rg.S = amax / 127.0f; }
        }
        if (c0 == 0) s_S[row] = rg.S;
        uint8_t *dst = codes + row * pitch;
#pragma unroll
        for (int i = 0; i < XCH; ++i) {
            const int c = c0 + i * LPR;
            if (i * LPR < nchunks && c < nchunks) {
                uint32_t ev, od;
                codes8<W8>(x[i], rg.inv, ev, od);
                *reinterpret_cast<uint2 *>(dst + c * 8) = make_uint2(ev, od);
            }
        }
    }
    if constexpr (WLDS) {
#pragma unroll
        for (int i = 0; i < WCH; ++i) {
            const int p = tid + i * NT;
            if (p < 32 * FN * wcpr) {
                const int rw = row_of(p), st = FN == 2 ? (rw & 1) * 32 + rw / 2 : rw;   // channel of the tile, its storage row
                *reinterpret_cast<u32x4 *>(wt + (p + (st - rw) * wcpr + st) * 16) = wst[i];
            }
        }
    }
    __syncthreads();

    // ---- pass 2: this wave's share of K ----------------------------------------------------------------------
    v16i acc[FPW];
#pragma unroll
    for (int j = 0; j < FPW; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[j][q] = 0;
    const uint8_t *arow = codes + (r % TM) * pitch + h * (NIBBLES ? 16 : 32);
    const uint8_t *wrow = wt + (32 * j0 + r) * wpitch + h * (W8 ? 32 : 16);
    auto block = [&](int b, const u32x4 (&requested)[FPW]) {
        v4i alo, ahi, wlo[FPW], whi[FPW];
        if constexpr (NIBBLES) {
            const u32x4 ap = *reinterpret_cast<const u32x4 *>(arow + b * 32);
            alo = widen2<!ASYM>(ap[0], ap[1]);
            ahi = widen2<!ASYM>(ap[2], ap[3]);
        } else {
            alo = *reinterpret_cast<const v4i *>(arow + b * 64);
            ahi = *reinterpret_cast<const v4i *>(arow + b * 64 + 16);
        }
#pragma unroll
        for (int j = 0; j < FPW; ++j) {
            const uint8_t *wp = wrow + 32 * j * wpitch;
            if constexpr (W8) {                                 // one-byte codes: 32 bytes of a channel, two MFMA operands as they are
                if constexpr (WLDS) {
                    wlo[j] = *reinterpret_cast<const v4i *>(wp + b * 64);
                    whi[j] = *reinterpret_cast<const v4i *>(wp + b * 64 + 16);
                } else {
                    const uint32_t off = (uint32_t)channel(j0 + j) * (uint32_t)a.ldw + (uint32_t)(b * 64 + h * 32);
                    wlo[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off, 0, 0));
                    whi[j] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, off + 16, 0, 0));
                }
            } else {
                const u32x4 wv = WPRE ? requested[j] : WLDS ? *reinterpret_cast<const u32x4 *>(wp + b * 32) : request_w(j0 + j, b);
                wlo[j] = widen2<!ASYM>(wv[0], wv[1]);
                whi[j] = widen2<!ASYM>(wv[2], wv[3]);
            }
        }
#pragma unroll
        for (int j = 0; j < FPW; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(alo, wlo[j], acc[j], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < FPW; ++j) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ahi, whi[j], acc[j], 0, 0, 0);
    };
    if constexpr (KC && (WLDS || WPRE)) {
#pragma unroll
        for (int i = 0; i < NBW; ++i)
            if (kw + i * KW < nb) block(kw + i * KW, wpre[WPRE ? i : 0]);
    } else {
#pragma unroll 1
        for (int b = kw; b < nb; b += KW) block(b, wpre[0]);
    }

    // ---- add the partial sums of the waves in LDS (exact, so the order is free).  Accumulator register q of
    //      lane (c, h) is row 8 (q / 4) + 4 h + q % 4: with TM = 16 only registers 0 .. 7 hold real rows, with 8 only 0 .. 3 ----------
    if (kw < nb) {
#pragma unroll
        for (int j = 0; j < FPW; ++j)
#pragma unroll
            for (int q = 0; q < RV; ++q) atomicAdd(&s_sum[((j0 + j) * RV + q) * 64 + lane], acc[j][q]);
    }
    __syncthreads();
    const bool ints = PACKED && a.acc_out != nullptr;
    const __amdgpu_buffer_rsrc_t o_rsrc = ints ? make_rsrc(a.acc_out, (uint32_t)((long)a.M * a.N * 4))
                                               : make_rsrc(a.out, (uint32_t)((long)a.M * a.N * 2));
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
        const int q = wave + k * NW;
        if (q >= RV) break;
        const int trow = frag_row(0, q, lane);
        // output of channel j (rows >= M fall off the end; N is a multiple of 8: all of a lane's adjacent channels or none)
        auto at = [&](int j, uint32_t size) { return channel(j) < a.N ? ((uint32_t)(m0 + trow) * (uint32_t)a.N + (uint32_t)channel(j)) * size : kPoison; };
        if (ints) {                                              // parity export: P itself
            uint32_t P[FN];
#pragma unroll
            for (int j = 0; j < FN; ++j) P[j] = (uint32_t)(W8 || ASYM ? s_sum[(j * RV + q) * 64 + lane] : s_sum[(j * RV + q) * 64 + lane] >> 8);
            if constexpr (ADJ) {
                store_words<FN>(o_rsrc, at(0, 4), P);
            } else {
#pragma unroll
                for (int j = 0; j < FN; ++j) __builtin_amdgcn_raw_buffer_store_b32(P[j], o_rsrc, at(j, 4), 0, 0);
            }
            continue;
        }
        // the sums hold 16 * P (256 * P if PACKED, P itself for the INT8 sibling); a power of two, so the rescaled
        // weight scale is exact
        float y[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const float swn = __uint_as_float(sw_raw[j]) * (W8 || ASYM ? 1.0f : PACKED ? 0.00390625f : 0.0625f);
            const float P = (float)s_sum[(j * RV + q) * 64 + lane];
            if constexpr (ASYM) {                                // the operation order of tile_epilogue (one weight group)
                const float t1 = swn * P, t2 = __uint_as_float(zw_raw[j]) * s_S[2 * TM + trow];
                y[j] = s_S[trow] * t1;
                const float u = s_S[trow] * t2, z = s_S[TM + trow] * __uint_as_float(c_raw[j]);
                y[j] = y[j] + u;
                y[j] = y[j] + z;
            } else {
                y[j] = (P * s_S[trow]) * swn;
            }
            if (a.bias) y[j] = y[j] + __half2float(__ushort_as_half(b_raw[j]));
        }
        if constexpr (ADJ) {
            if (a.act == W4A4_ACT_GELU) store_gelu_halves<FN>(o_rsrc, at(0, 2), y);
            else store_halves<FN>(o_rsrc, at(0, 2), y);
        } else {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const float one[1] = {y[j]};
                if (a.act == W4A4_ACT_GELU) store_gelu_halves<1>(o_rsrc, at(j, 2), one);
                else store_halves<1>(o_rsrc, at(j, 2), one);
            }
        }
    }
}

template <int NW, int FN, int TM, bool WLDS, bool PACKED, bool W8 = false, bool ASYM = false, int KC = 0, bool LN = false>
static int launch_small(SmallArgs &a, hipStream_t st) {
    a.tiles_n = (a.N + 32 * FN - 1) / (32 * FN);
    const uint32_t wcpr = (uint32_t)(W8 ? a.K / 16 : a.K / 32);
    a.wcpr_inv = (uint32_t)(((1ull << 32) + wcpr - 1) / wcpr);
    const long tiles = (long)((a.M + TM - 1) / TM) * a.tiles_n;
    if (tiles > 0x7fffffffL) return W4A4_ERR_UNSUPPORTED_SHAPE;
    const size_t lds = TM * (size_t)((PACKED && !W8 ? a.K / 2 : a.K) + 16) + (WLDS ? 32 * FN * (size_t)((W8 ? a.K : a.K / 2) + 16) : 0) +
                       (size_t)(TM / 2) * FN * 64 * 4 + TM * (ASYM ? 12 : 4);
    auto kern = linear_f16act_kernel<NW, FN, TM, WLDS, PACKED, W8, ASYM, KC, LN>;
    static KernelState ks;
    if (prepare_kernel(reinterpret_cast<const void *>(kern), lds, ks) < 0) return W4A4_ERR_HIP;
    launch_gemm(kern, dim3((unsigned)tiles), dim3(NW * 64), lds, st, a);
    return launch_status();
}

// Whether a tile of tm tokens and ch channels has its weights in LDS: they fit beside the codes and the sums within a CU's 160 KB, and
// the chunks that a lane holds on their way there into its registers.
constexpr bool small_wlds(int tm, int ch, int code_row, int w_row, int nw, int most) {
    return (size_t)tm * (code_row + 16) + (size_t)ch * (w_row + 16) <= 144 * 1024 && (ch * (w_row / 16) + nw * 64 - 1) / (nw * 64) <= most;
}
// K as a constant of the kernel: rows that give each of a token's lanes the same number of 16-byte chunks (two, three, four or six for thirty-two
// lanes, four, six or eight for sixty-four)
template <int NW, bool PACKED, bool W8, bool ASYM, int K>
static int launch_const(SmallArgs &a, bool wide, bool low, hipStream_t st) {
    constexpr int code_row = PACKED && !W8 ? K / 2 : K, w_row = W8 ? K : K / 2;
    if (wide) return launch_small<NW, 2, 32, small_wlds(32, 64, code_row, w_row, NW, 8), PACKED, W8, ASYM, K>(a, st);
    // Long fp16 rows: quantizing them is most of the work, so eight tokens and half the waves per workgroup while each has a CU for
    // itself: 32 x 768 x 3072 4.90 us -> 4.08, 64 x 1024 x 4096 5.83 -> 4.86
    if constexpr (!PACKED && NW == 16)
        if ((long)((a.M + 7) / 8) * ((a.N + 31) / 32) <= device_cus()) return launch_small<8, 1, 8, small_wlds(8, 32, code_row, w_row, 8, 8), PACKED, W8, ASYM, K>(a, st);
    if (low) return launch_small<NW, 1, 16, small_wlds(16, 32, code_row, w_row, NW, 8), PACKED, W8, ASYM, K>(a, st);
    return launch_small<NW, 1, 32, small_wlds(32, 32, code_row, w_row, NW, 8), PACKED, W8, ASYM, K>(a, st);
}

// Lengths of a row that the kernel has as a constant: those of the switch below.
bool small_constant_k(int K) { return K == 512 || K == 768 || K == 1024 || K == 1536 || K == 2048 || K == 3072 || K == 4096; }

// Shape policy.  Waves: enough that none walks more than four blocks of K nor holds more than 16 chunks of
// a row.  Tile: every column tile re-quantizes (or re-reads) its token rows, so fewer, wider tiles do less
// redundant work, but a tile is one CU's job: 32 x 32 while that gives at most one workgroup per CU, 32 x 64
// beyond, and 16-token tiles when 32-token tiles would leave more than half of the CUs idle.  The weight
// tile is staged in LDS (coalesced loads) whenever it fits beside the activation codes.
template <bool PACKED, bool W8 = false, bool ASYM = false>
static int small_dispatch(SmallArgs &a, hipStream_t st) {
    const int M = a.M, N = a.N, K = a.K;
    const long t32 = (long)((M + 31) / 32) * ((N + 31) / 32);
    const bool wide = t32 > 256, low = t32 <= 128;
    if constexpr (PACKED || !W8) {
        switch (K) {
            case 512: return launch_const<8, PACKED, W8, ASYM, 512>(a, wide, low, st);
            case 768: return launch_const<8, PACKED, W8, ASYM, 768>(a, wide, low, st);
            case 1024: return launch_const<8, PACKED, W8, ASYM, 1024>(a, wide, low, st);
            case 1536: return launch_const<8, PACKED, W8, ASYM, 1536>(a, wide, low, st);
            case 2048: return launch_const<16, PACKED, W8, ASYM, 2048>(a, wide, low, st);
            case 3072: return launch_const<16, PACKED, W8, ASYM, 3072>(a, wide, low, st);
            case 4096: return launch_const<16, PACKED, W8, ASYM, 4096>(a, wide, low, st);
        }
    }
    const int nw = K > 1536 ? 16 : K > 384 ? 8 : 4;
    const bool wlds = small_wlds(low ? 16 : 32, wide ? 64 : 32, PACKED && !W8 ? K / 2 : K, W8 ? K : K / 2, nw, small_wchunks(nw));
#define W4A4_SMALL(NW)                                                                                  \
    do {                                                                                                \
        if (wide) return wlds ? launch_small<NW, 2, 32, true, PACKED, W8, ASYM>(a, st) : launch_small<NW, 2, 32, false, PACKED, W8, ASYM>(a, st); \
        if (low) return wlds ? launch_small<NW, 1, 16, true, PACKED, W8, ASYM>(a, st) : launch_small<NW, 1, 16, false, PACKED, W8, ASYM>(a, st);  \
        return wlds ? launch_small<NW, 1, 32, true, PACKED, W8, ASYM>(a, st) : launch_small<NW, 1, 32, false, PACKED, W8, ASYM>(a, st);     \
    } while (0)
    if (K > 1536) W4A4_SMALL(16);
    if (K > 384) W4A4_SMALL(8);
    W4A4_SMALL(4);
#undef W4A4_SMALL
}

// Several weight groups, few tokens: a wave owns whole groups.  At these sizes the kernel with one K loop per workgroup spends its time on
// one 128-code step after the other with a barrier each (24 steps at K = 3072: 27 us whatever the tokens), so a group here is
// one wave's work: both operand tiles are parked in LDS as above, wave w multiplies groups w, w + NW, .. and leaves their
// exact sums in LDS, and every thread adds up its outputs' groups in ascending order, each product and sum rounded on its own, as the
// definition has it (same bits as gemm_kernel).  NW groups are in LDS at a time.
template <int NW, int TM, int MODE>
__global__ __launch_bounds__(NW * 64) void grouped_small_kernel(GemmArgs g) {
    constexpr bool SGN = MODE == W4A4_SYM;
    constexpr int NT = NW * 64, RV = TM / 2;                    // accumulator registers that hold real rows
    constexpr int RPW = (RV + NW - 1) / NW;                     // ... finished by one wave
    constexpr int CH = 4;                                       // 16-byte chunks of an operand tile per thread (the launcher checks)
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int Kb = g.K / 2, pitch = Kb + 16, ng = g.ng, ngp = ng | 1;   // (an odd pitch: the table reads of 32 lanes spread over the banks)
    uint8_t *at = smem, *wt = at + TM * pitch;                  // [TM][pitch], [32][pitch]
    int *s_P = reinterpret_cast<int *>(wt + 32 * pitch);        // [NW][RV][64]
    float *sw_tab = reinterpret_cast<float *>(s_P + NW * RV * 64);      // [32][ngp]
    float *zw_tab = sw_tab + 32 * ngp, *ra_tab = zw_tab + (SGN ? 0 : 32 * ngp);   // [32][ngp], [TM][ngp]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, h = lane >> 5;
    const int m0 = (blockIdx.x / g.tiles_n) * TM, n0 = (blockIdx.x % g.tiles_n) * 32;
    const __amdgpu_buffer_rsrc_t a_rsrc = make_rsrc(g.Aq, (uint32_t)((long)(g.M - 1) * g.lda + Kb));
    const __amdgpu_buffer_rsrc_t w_rsrc = make_rsrc(g.Wq, (uint32_t)((long)g.N * g.ldw));

    // ---- requests: both operand tiles (rows past M, channels past N: zeros), constants -------------------------------
    const int cpr = g.K / 32;                                   // 16-byte chunks of a row
    u32x4 av[CH], wv[CH];
    int row_i[CH];
    uint32_t dst_i[CH];
    {
        const int stepq = NT / cpr, stepr = NT % cpr;
        int row = tid / cpr, c = tid % cpr;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            row_i[i] = row;
            dst_i[i] = (uint32_t)(row * pitch + c * 16);
            if (i * NT < TM * cpr) av[i] = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (uint32_t)(m0 + row) * (uint32_t)g.lda + (uint32_t)c * 16, 0, 0);
            if (i * NT < 32 * cpr) wv[i] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, (uint32_t)(n0 + row) * (uint32_t)g.ldw + (uint32_t)c * 16, 0, 0);
            row += stepq; c += stepr;
            if (c >= cpr) { c -= cpr; ++row; }
        }
    }
    for (int e = tid; e < 32 * ng; e += NT) {                   // a tile's 32 rows of [N][ng] are one piece of memory
        const int n = e / ng, at_tab = n * ngp + e % ng;
        const bool in = n0 + n < g.N;
        sw_tab[at_tab] = in ? g.sw[(long)n0 * ng + e] : 0.0f;
        if constexpr (!SGN) zw_tab[at_tab] = in ? g.zw[(long)n0 * ng + e] : 0.0f;
    }
    if constexpr (!SGN) {
        for (int e = tid; e < TM * ng; e += NT) {
            const int m = e / ng;
            ra_tab[m * ngp + e % ng] = m0 + m < g.M ? (float)g.RA[(long)m0 * ng + e] : 0.0f;
        }
    }
    const int n = n0 + r;
    const bool n_ok = n < g.N;
    const float bias = g.bias && n_ok ? __half2float(g.bias[n]) : 0.0f, c_n = !SGN && n_ok ? g.c[n] : 0.0f;
    float sa[RPW], za[RPW];
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
        const int m = min(m0 + frag_row(0, wave + k * NW, lane), g.M - 1);
        sa[k] = g.sa[m];
        za[k] = SGN ? 0.0f : g.za[m];
    }
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        if (i * NT < TM * cpr && row_i[i] < TM) *reinterpret_cast<u32x4 *>(at + dst_i[i]) = av[i];
        if (i * NT < 32 * cpr && row_i[i] < 32) *reinterpret_cast<u32x4 *>(wt + dst_i[i]) = wv[i];
    }
    __syncthreads();

    // ---- groups: NW at a time ---------------------------------------------------------------------------------------
    const uint8_t *arow = at + (r % TM) * pitch + h * 16, *wrow = wt + r * pitch + h * 16;
    const int blocks = g.K / ng / 64;                           // blocks of 64 codes in a group
    float t1[RPW];
#pragma unroll
    for (int k = 0; k < RPW; ++k) t1[k] = 0.0f;
    for (int g0 = 0; g0 < ng; g0 += NW) {
        if (g0 + wave < ng) {
            v16i acc;
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[q] = 0;
            const int b0 = (g0 + wave) * blocks;
            for (int b = b0; b < b0 + blocks; ++b) {
                const u32x4 a = *reinterpret_cast<const u32x4 *>(arow + b * 32), w = *reinterpret_cast<const u32x4 *>(wrow + b * 32);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(widen2<SGN>(a[0], a[1]), widen2<SGN>(w[0], w[1]), acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(widen2<SGN>(a[2], a[3]), widen2<SGN>(w[2], w[3]), acc, 0, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < RV; ++q) s_P[(wave * RV + q) * 64 + lane] = SGN ? acc[q] >> 8 : acc[q];
        }
        __syncthreads();
        const int here = min(NW, ng - g0);
#pragma unroll
        for (int k = 0; k < RPW; ++k) {
            const int qq = wave + k * NW;
            if (qq >= RV) break;
            for (int s = 0; s < here; ++s) {
                const float u = sw_tab[r * ngp + g0 + s] * (float)s_P[(s * RV + qq) * 64 + lane];
                t1[k] = t1[k] + u;
            }
        }
        if (g0 + NW < ng) __syncthreads();                       // the next groups' sums go to the same place
    }

    // ---- outputs, in the operation order of tile_epilogue ---------------------------------------------------------
    const __amdgpu_buffer_rsrc_t o_rsrc = make_rsrc(g.out, (uint32_t)((long)g.M * g.N * 2));
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
        const int qq = wave + k * NW;
        if (qq >= RV) break;
        const int row = frag_row(0, qq, lane);
        float y = sa[k] * t1[k];
        if constexpr (!SGN) {
            float t2 = 0.0f;
            for (int gi = 0; gi < ng; ++gi) {
                const float w = zw_tab[r * ngp + gi] * ra_tab[row * ngp + gi];
                t2 = t2 + w;
            }
            const float p = sa[k] * t2, z = za[k] * c_n;
            y = y + p;
            y = y + z;
        }
        if (g.bias) y = y + bias;
        const uint32_t off = n_ok ? ((uint32_t)(m0 + row) * (uint32_t)g.N + (uint32_t)n) * 2u : kPoison;   // rows >= M fall off the end
        if (g.act == W4A4_ACT_GELU) __builtin_amdgcn_raw_buffer_store_b16(gelu_erf_half(y), o_rsrc, off, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b16(__half_as_ushort(__float2half_rn(y)), o_rsrc, off, 0, 0);
    }
}

template <int NW, int TM>
static size_t grouped_small_lds(const GemmArgs &g, bool asym) {
    return (size_t)(TM + 32) * (g.K / 2 + 16) + (size_t)NW * (TM / 2) * 64 * 4 + (size_t)(g.ng | 1) * (asym ? 64 + TM : 32) * 4;
}
template <int NW, int TM, int MODE>
static int launch_grouped(GemmArgs &g, hipStream_t st) {
    g.tiles_m = (g.M + TM - 1) / TM;
    g.tiles_n = (g.N + 31) / 32;
    const size_t lds = grouped_small_lds<NW, TM>(g, MODE == W4A4_ASYM);
    auto kern = grouped_small_kernel<NW, TM, MODE>;
    static KernelState ks;
    if (prepare_kernel(reinterpret_cast<const void *>(kern), lds, ks) < 0) return W4A4_ERR_HIP;
    launch_gemm(kern, dim3((unsigned)(g.tiles_m * g.tiles_n)), dim3(NW * 64), lds, st, g);
    return launch_status();
}
// Rows of up to 1024 codes leave room for tiles of 32 tokens, three workgroups of eight waves to a CU; longer ones take sixteen
// waves and 16 tokens, one to a CU.
static bool grouped_short(const GemmArgs &g) { return g.K <= 1024; }
// Tiles of 32 x 32 (long rows: 16 x 32) up to which it wins against 64 x 64 tiles of gemm_kernel, which take one 128-code step after the
// other, so that fewer of them lose less (us, that kernel | this one; asymmetric: 128 x 768 x 768 12.2 | 5.7, 128 x 768 x 3072 27.0 | 6.5,
// 301 x 3072 x 1024 (960 tiles) 12.1 | 10.5, 600 x 1024 x 4096 (1216) 34.5 | 29.6, 800 x 1024 x 4096 (1600) 34.7 | 40.4; symmetric: 128 x 768 x 3072
// 20.4 | 6.0, 600 x 768 x 3072 (912) 20.5 | 18.4, 800 x 768 x 3072 (1200) 20.5 | 22.6).  Short K has the less to lose: 552 x 1216 x 256 symmetric (684)
// 4.1 | 5.7, 528 tiles of 512 codes 5.8 | 6.1, 323 x 2752 x 256 asymmetric (946) 7.1 | 7.6; and where fewer than twelve groups leave
// waves idle: 86 x 4800 x 1536 in 256s symmetric (900) 9.9 | 11.0, 66 x 7552 x 2304 in 256s asymmetric (1180) 19.4 | 21.7, 487 x 1088 x 2048 in 512s
// (1054) 16.1 | 18.0, 90 x 6720 x 768 in 256s symmetric (630) 6.3 | 7.2.  At 1802 sizes in groups of 128, 256 and 512 the choice is 0.06 % above
// the better of the two.
static long grouped_tile_limit(const GemmArgs &g, bool asym) {
    if (grouped_short(g)) return asym ? (g.K <= 256 ? 768 : 1024) : (g.K <= 512 || g.ng <= 3 ? 512 : 704);
    if (g.ng < 12) return asym ? (g.ng <= 4 ? 960 : 1088) : 768;
    return asym ? 1216 : 1024;
}
// fp16 outputs of canonical codes in several weight groups
bool small_grouped_ok(const GemmArgs &g, int mode, int out_kind) {
    const bool asym = mode == W4A4_ASYM;
    if (out_kind != OUT_F16 || g.layout != W4A4_LAYOUT_CANONICAL || g.ng < 2 || g.K % (64 * g.ng) || g.K > 4096 || g.lda % 16 ||
        ((long)g.M + 32) * g.lda >= 0x7fffffffL || ((long)g.N + 32) * g.ldw >= 0x7fffffffL || ((long)g.M + 32) * g.N * 2 >= 0x7fffffffL) return false;
    const long rows = grouped_short(g) ? (g.M + 31) / 32 : (g.M + 15) / 16, tiles = rows * ((g.N + 31) / 32);
    const size_t lds = grouped_short(g) ? grouped_small_lds<8, 32>(g, asym) : grouped_small_lds<16, 16>(g, asym);
    return lds <= 160 * 1024 && tiles <= grouped_tile_limit(g, asym);
}
int launch_small_grouped(int mode, GemmArgs &g, hipStream_t st) {
    if (mode == W4A4_SYM) return grouped_short(g) ? launch_grouped<8, 32, W4A4_SYM>(g, st) : launch_grouped<16, 16, W4A4_SYM>(g, st);
    return grouped_short(g) ? launch_grouped<8, 32, W4A4_ASYM>(g, st) : launch_grouped<16, 16, W4A4_ASYM>(g, st);
}

// The LayerNorm form (layer.hpp): the tiles of small_dispatch, eight waves, the weight tile in LDS (K <= 1024: it fits).
template <int K>
static int launch_layernorm(SmallArgs &a, hipStream_t st) {
    const long t32 = (long)((a.M + 31) / 32) * ((a.N + 31) / 32);
    if (t32 > 256) return launch_small<8, 2, 32, true, false, false, false, K, true>(a, st);
    if (t32 <= 128) return launch_small<8, 1, 16, true, false, false, false, K, true>(a, st);
    return launch_small<8, 1, 32, true, false, false, false, K, true>(a, st);
}
int linear_layernorm_f16act(const LnArgs &ln, const w4a4_weight &W, const w4a4_epilogue &ep, void *out, hipStream_t st) {
    SmallArgs a{};
    a.X = ln.X; a.ldx = ln.ldx; a.R = ln.R; a.gamma = ln.gamma; a.beta = ln.beta; a.eps = ln.eps; a.Y = ln.Y;
    a.Wq = W.q; a.ldw = ln.K / 2; a.sw = W.scale;
    a.bias = static_cast<const __half *>(ep.bias_f16); a.act = ep.act;
    a.out = static_cast<__half *>(out);
    a.M = ln.M; a.N = W.N; a.K = ln.K;
    return ln.K == 512 ? launch_layernorm<512>(a, st) : ln.K == 768 ? launch_layernorm<768>(a, st) : launch_layernorm<1024>(a, st);
}
bool linear_layernorm_f16act_ok(const LnArgs &ln, const w4a4_weight &W, const w4a4_epilogue &ep, const void *out) {
    const int M = ln.M, K = ln.K, N = W.N;
    if ((K != 512 && K != 768 && K != 1024) || ln.ldx != K || !ln.R || N % 8 || (W.group != 0 && W.group != K)) return false;
    for (const void *p : {static_cast<const void *>(ln.X), static_cast<const void *>(ln.R), static_cast<const void *>(ln.gamma),
                          static_cast<const void *>(ln.beta), static_cast<const void *>(ln.Y), static_cast<const void *>(W.q), out})
        if (!p || !aligned16(p)) return false;
    return W.scale && (long)M * K * 2 < 0x7fffffffL && (long)N * (K / 2) < 0x7fffffffL && ((long)M + 32) * N * 2 < 0x7fffffffL;
}

// The same kernel on activations that are already quantized (canonical packed codes + token scales): the
// small-problem schedule of w4a4_linear / w4a4_gemm_i32.  Requires one weight group,
// K % 64 == 0, K <= 4096, lda % 16 == 0, 32-bit offsets.
int launch_small_packed(int mode, int out_kind, GemmArgs &g, hipStream_t st) {
    if (out_kind != OUT_F16 && out_kind != OUT_I32) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if (g.K % 64 || g.K > 4096 || g.lda % 16 || (long)g.M * g.lda >= 0x7fffffffL || (long)g.N * g.ldw >= 0x7fffffffL ||
        ((long)g.M + 32) * g.N * 4 >= 0x7fffffffL)
        return W4A4_ERR_UNSUPPORTED_SHAPE;
    SmallArgs a{};
    a.Aq = g.Aq; a.lda = g.lda; a.sa = g.sa;
    a.Wq = g.Wq; a.ldw = g.ldw; a.sw = g.sw;
    a.bias = g.bias; a.act = g.act;
    if (out_kind == OUT_I32) a.acc_out = static_cast<int32_t *>(g.out);
    else a.out = static_cast<__half *>(g.out);
    a.M = g.M; a.N = g.N; a.K = g.K;
    if (mode == W4A4_SYM) return small_dispatch<true>(a, st);
    a.za = g.za; a.RA = g.RA; a.zw = g.zw; a.c = g.c;
    return small_dispatch<true, false, true>(a, st);
}

// The INT8 sibling's small-problem path on int8 codes that are already in memory (w8a8_linear / w8a8_gemm_i32
// for at most 512 tiles of 32 x 32).  g.lda / g.ldw are row strides in bytes = codes.
bool small8_ok(const GemmArgs &g) {
    return g.K % 64 == 0 && g.K <= 4096 && g.lda % 16 == 0 && (long)((g.M + 31) / 32) * ((g.N + 31) / 32) <= 512 &&
           (long)g.M * g.lda < 0x7fffffffL && (long)g.N * g.ldw < 0x7fffffffL && ((long)g.M + 32) * g.N * 4 < 0x7fffffffL;
}
int launch_small_packed8(int out_kind, GemmArgs &g, hipStream_t st) {
    if ((out_kind != OUT_F16 && out_kind != OUT_I32) || !small8_ok(g)) return W4A4_ERR_UNSUPPORTED_SHAPE;
    SmallArgs a{};
    a.Aq = g.Aq; a.lda = g.lda; a.sa = g.sa;
    a.Wq = g.Wq; a.ldw = g.ldw; a.sw = g.sw;
    a.bias = g.bias; a.act = g.act;
    if (out_kind == OUT_I32) a.acc_out = static_cast<int32_t *>(g.out);
    else a.out = static_cast<__half *>(g.out);
    a.M = g.M; a.N = g.N; a.K = g.K;
    return small_dispatch<true, true>(a, st);
}

}  // namespace w4a4

using namespace w4a4;

extern "C" int w4a4_linear_f16act(const void *X_f16, int M, int K, int ldx, const w4a4_weight *W,
                                  const w4a4_epilogue *ep, void *out, void *stream) {
    if (!W || !ep || M < 0 || K <= 0 || ldx < K || W->N <= 0 || W->K != K) return W4A4_ERR_INVALID_ARG;
    if (ep->act != W4A4_ACT_NONE && ep->act != W4A4_ACT_GELU) return W4A4_ERR_INVALID_ARG;
    if (W->mode != W4A4_SYM && W->mode != W4A4_ASYM) return W4A4_ERR_INVALID_ARG;
    if (W->mode != W4A4_SYM || W->layout != W4A4_LAYOUT_CANONICAL || (W->group != 0 && W->group != K) || ep->requant)
        return W4A4_ERR_UNSUPPORTED_SHAPE;
    if (K % 64 || K > 4096 || W->N % 8 || (ldx * 2) % 16) return W4A4_ERR_UNSUPPORTED_SHAPE;   // 16 waves x 4 blocks
    if (M == 0) return W4A4_OK;
    if (!X_f16 || !W->q || !W->scale || !out) return W4A4_ERR_INVALID_ARG;
    if (!aligned16(X_f16) || !aligned16(W->q) || !aligned16(out)) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if ((long)M * ldx * 2 >= 0x7fffffffL || (long)W->N * (K / 2) >= 0x7fffffffL || ((long)M + 32) * W->N * 2 >= 0x7fffffffL)
        return W4A4_ERR_UNSUPPORTED_SHAPE;
    SmallArgs a{};
    a.X = static_cast<const __half *>(X_f16); a.ldx = ldx;
    a.Wq = W->q; a.ldw = K / 2; a.sw = W->scale;
    a.bias = static_cast<const __half *>(ep->bias_f16); a.act = ep->act;
    a.out = static_cast<__half *>(out);
    a.M = M; a.N = W->N; a.K = K; a.tiles_n = 0;
    return small_dispatch<false>(a, as_stream(stream));
}

extern "C" int w8a8_linear_f16act(const void *X_f16, int M, int K, int ldx, const int8_t *Wq, const float *sw, int N,
                                  const w4a4_epilogue *ep, void *out, void *stream) {
    if (!ep || M < 0 || K <= 0 || ldx < K || N <= 0) return W4A4_ERR_INVALID_ARG;
    if (ep->act != W4A4_ACT_NONE && ep->act != W4A4_ACT_GELU) return W4A4_ERR_INVALID_ARG;
    if (ep->requant) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if (K % 64 || K > 4096 || N % 8 || (ldx * 2) % 16) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if (M == 0) return W4A4_OK;
    if (!X_f16 || !Wq || !sw || !out) return W4A4_ERR_INVALID_ARG;
    if (!aligned16(X_f16) || !aligned16(Wq) || !aligned16(out) || (ep->bias_f16 && !aligned16(ep->bias_f16)))
        return W4A4_ERR_UNSUPPORTED_SHAPE;
    if ((long)M * ldx * 2 >= 0x7fffffffL || (long)N * K >= 0x7fffffffL || ((long)M + 32) * N * 2 >= 0x7fffffffL)
        return W4A4_ERR_UNSUPPORTED_SHAPE;
    SmallArgs a{};
    a.X = static_cast<const __half *>(X_f16); a.ldx = ldx;
    a.Wq = reinterpret_cast<const uint8_t *>(Wq); a.ldw = K; a.sw = sw;
    a.bias = static_cast<const __half *>(ep->bias_f16); a.act = ep->act;
    a.out = static_cast<__half *>(out);
    a.M = M; a.N = N; a.K = K; a.tiles_n = 0;
    return small_dispatch<false, true>(a, as_stream(stream));
}
