// Persistent GEMM for asymmetric layers in weight groups of 128 codes on unsigned codes kept in the MFMA operand layout (see
// w4a4_layout), K a multiple of 128, K >= 640:
//     t1[m,n] = sum_g sw[n,g] * P_g[m,n],      P_g = sum_{k in g} qa[m,k] * qw[n,k]
//     y       = sa[m]*(t1 + sum_g zw[n,g]*RA[m,g]) + za[m]*c[n] + bias[n]
//
// What bounds it is the vector ALU: the sums of every group have to be scaled before they may be added up, and the nibbles have to
// become matrix operands.  So the codes go to the matrix cores as FP8: the byte 0x0u read as E4M3 is u * 2^-9 for every u in 0 .. 15
// (eight subnormals and the first binade, both in steps of 2^-9), its products are multiples of 2^-18, and their sum, kept in FP32, is
// exact (225 * 128 < 2^24).  Against int8 operands (one v_and per register, accumulators holding 16*(P_g - 8*AE - 8*WO)) that
//   * takes the conversion to float out of the fold, which is ONE fused multiply-add per accumulator and group,
//     t1 = fma(sw[n,g] * 2^18, acc, t1), for half an instruction more per operand register (the nibble that the layout keeps
//     shifted up by four and minus 8 needs a shift, and a mask with an exclusive or);
//   * needs no token and channel terms AE, WO: the first MFMAs of a group start from the constant zero;
//   * takes half as many matrix instructions, of 64 codes each (the same time: FP8 runs at the rate of int8).
// The fold is spread over the slots of the next group's first MFMAs, fragment k in front of the MFMA that starts it anew, while
// the one before it runs, and so is the zero-point sum, a rank-ng product by the fp32 MFMA, which cost 6 of 57 us in the
// epilogue of 24 groups, as a loop over tables in LDS.
// int8 operands, folds and zero points behind the MFMAs | this (us): 16384 x 2304 x 768 50.4 | 45.4, 16384 x 768 x 768 19.3 | 17.9,
// 16384 x 3072 x 768 + GELU 80.0 | 74.5, 16384 x 768 x 3072 56.8 | 50.0, 4096 x 768 x 3072 25.0 | 22.2.  Left of the last but one: 8 us are
// the zero-point sum, 8 the tiles' way through LDS, 11 the folds, which two waves per SIMD do not hide from each other.
//   * Tiles travel HBM -> LDS by `buffer_load_dwordx4 ... lds` with scalar addressing, unpadded LDS rows with an XOR swizzle, four stages
//     (three: 16384 x 768 x 3072 51.5, 4096 x 768 x 3072 23.9), persistent workgroups whose K steps form one stream across tiles.
//   * 128 x 128 tiles, four waves of 64 x 64 (64 accumulators of the group and 64 of t1 per lane), two workgroups per CU.
//   * Token scales and zero points go to LDS by 4-byte DMA; the scales of a channel's groups and the entries of the zero-point tables are
//     fetched into registers, four groups to a request: one whose 64 lanes touch 32 or 64 cache lines occupies the memory path of the CU
//     for as many cycles.
// With 32 groups the order of the sum decides its rounding noise; here the groups' sums (t1) and the zero-point sum (minus t1, nearly) grow
// side by side, and the partial sums stay small.
#include "gemm_common.hpp"

namespace w4a4 {

typedef __attribute__((address_space(3))) void *lds_ptr_t;
typedef int v8i __attribute__((ext_vector_type(8)));

// s_waitcnt immediate for "vmcnt <= n and lgkmcnt == 0", expcnt unconstrained (gfx9 encoding)
static constexpr int vmcnt_and_lds(int n) { return (n & 0xF) | (0x7 << 4) | (0x0 << 8) | (((n >> 4) & 0x3) << 14); }
// ... for "lgkmcnt == 0", vmcnt unconstrained
static constexpr int lds_only() { return 0xC07F; }
// ... for "vmcnt <= n", lgkmcnt and expcnt unconstrained
static constexpr int vmcnt_only(int n) { return (n & 0xF) | (0x7 << 4) | (0xF << 8) | (((n >> 4) & 0x3) << 14); }

// 32 codes of a row as FP8: words of four codes, positions 8i + 0, 2, 4, 6 and 8i + 1, 3, 5, 7 in turn, the same of either operand.
// Activations keep the even positions in the low nibbles and the odd ones, minus 8, in the high nibbles; weights the reverse.
__device__ __forceinline__ int fp8_low(uint32_t x) { return (int)(x & 0x0F0F0F0Fu); }
__device__ __forceinline__ int fp8_high(uint32_t x) { return (int)(((x >> 4) & 0x0F0F0F0Fu) ^ 0x08080808u); }

// NS: LDS stages.
template <int OUT, int NS>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
void gemm_group_olay_kernel(GemmArgs g) {
    constexpr int FM = 2, FN = 2, WM = 2, WN = 2;
    constexpr int BM = WM * FM * 32, BN = WN * FN * 32, NW = WM * WN;
    constexpr int ROWB = 64;                                    // bytes of a row per K step: the 128 codes of a group
    constexpr int SUB = ROWB / 32;                              // sub-steps of 64 codes
    constexpr int CPR = ROWB / 16, RPB = 1024 / ROWB;           // 16-byte chunks of a row, rows of a 1 KB DMA block
    constexpr int SWZ = 2;                                      // rows that share a swizzle, log2: 256 bytes of LDS
    constexpr int STAGE = (BM + BN) * ROWB;
    constexpr int LD = (BM + BN) / RPB / NW;                    // tile DMA instructions per wave per stage
    constexpr int A_LD = (BM / RPB) / NW;                       // the first A_LD of them fetch activations
    constexpr int NF = FM + FN, NM = FM * FN;
    static_assert(NF <= NM && LD <= 2 * NM, "not enough MFMA slots to hide the memory operations");

    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    uint8_t *par = smem + NS * STAGE;                           // [2 parities][ sa[BM] | za[BM] ]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int total = g.tiles_m * g.tiles_n, stride = gridDim.x;
    const int KT = g.K / (2 * ROWB);                            // K steps of a tile = groups, at least NS

    // ---- global -> LDS plan (fixed for the whole kernel) -------------------------------------------
    // DMA instruction i of this wave fills block wave + i*NW of a stage, rows RPB (wave + i*NW) ..: what i adds is the same for
    // all lanes (and leaves the swizzle alone).  LDS row p of the weight tile holds output channel nl: MFMA column cc of fragment f
    // is channel cc*FN + f of the wave's span, so a lane ends up with FN adjacent channels.
    constexpr int STRIDE = NW * RPB;                            // rows from one instruction to the next: 32 or 64
    static_assert(STRIDE % 32 == 0 && FN == 2, "whole fragments, two to a span");
    const int row0 = wave * RPB + lane / CPR, chunk = (lane % CPR) ^ ((row0 >> SWZ) & (CPR - 1));
    const int voff_a = row0 * (int)g.lda + chunk * 16;
    const int voff_b = ((row0 % 32) * FN + row0 / 32) * (int)g.ldw + chunk * 16;
    auto dma_voff = [&](int i) {                                // (added where it is needed, to the vector offset, since the scalar
        int v = i < A_LD ? voff_a : voff_b;                     //  one carries K; not a sum to keep in a register for the whole
        asm volatile("" : "+v"(v));                             //  loop)
        if (i < A_LD) return v + i * STRIDE * (int)g.lda;
        const int p = (i - A_LD) * STRIDE;
        return v + (p / 64 * 64 + p % 64 / 32) * (int)g.ldw;
    };
    // (exists == false: no bytes at all, so that the prefetch of a tile that does not exist touches no memory)
    auto a_desc = [&](int m0, bool exists = true) {
        const int rows = min(BM, g.M - m0);
        return make_rsrc(g.Aq + (long)m0 * g.lda, exists ? (uint32_t)((long)(rows - 1) * g.lda + g.K / 2) : 0u);
    };
    auto b_desc = [&](int n0, bool exists = true) {
        const int rows = min(BN, g.N - n0);
        return make_rsrc(g.Wq + (long)n0 * g.ldw, exists ? (uint32_t)((long)rows * g.ldw) : 0u);
    };
    auto dma4 = [&](__amdgpu_buffer_rsrc_t rs, void *dst, int vo) {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass only needs the kernel's signature; it rejects the LDS cast
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)dst, 4, vo, 0, 0, 0);
#else
        (void)rs; (void)dst; (void)vo;
#endif
    };
    auto dma_one = [&](int i, int stage, __amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb, int so) {
        uint8_t *dst = smem + stage * STAGE + (wave + i * NW) * 1024;
#if defined(__HIP_DEVICE_COMPILE__)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(i < A_LD ? ra : rb, (lds_ptr_t)dst, 16, dma_voff(i), so, 0, 0);
#else
        (void)dst; (void)ra; (void)rb; (void)so;
#endif
    };
    const __amdgpu_buffer_rsrc_t sa_rsrc = make_rsrc(g.sa, (uint32_t)g.M * 4u);
    const __amdgpu_buffer_rsrc_t za_rsrc = make_rsrc(g.za, (uint32_t)g.M * 4u);
    const __amdgpu_buffer_rsrc_t sw_rsrc = make_rsrc(g.sw, (uint32_t)((long)g.N * g.ng * 4));
    const __amdgpu_buffer_rsrc_t zw_rsrc = make_rsrc(g.zw, (uint32_t)((long)g.N * g.ng * 4));
    const __amdgpu_buffer_rsrc_t ra_rsrc = make_rsrc(g.RA, (uint32_t)((long)g.M * g.ng * 4));
    const __amdgpu_buffer_rsrc_t c_rsrc = make_rsrc(g.c, (uint32_t)g.N * 4u);
    const __amdgpu_buffer_rsrc_t bias_rsrc = make_rsrc(g.bias, g.bias ? (uint32_t)g.N * 2u : 0u);   // no bias: zeros
    // Token scales and zero points of a tile, double buffered by parity; 64 values per DMA instruction, one per wave.
    auto dma_tokens = [&](int m0, int parity) {
        const bool is_sa = wave < 2;
        dma4(is_sa ? sa_rsrc : za_rsrc, par + parity * (2 * BM * 4) + (is_sa ? 0 : BM * 4) + (wave & 1) * 256, (m0 + (wave & 1) * 64 + lane) * 4);
    };
    // ---- operand fragments -----------------------------------------------------------------------
    const int swz = ((lane & 31) >> SWZ) & (CPR - 1);
    const int rd0 = (lane & 31) * ROWB + (((lane >> 5) ^ swz) << 4);   // sub-step 0;  sub-step ss is rd0 ^ (32 * ss)
    int frag_off[NF];
#pragma unroll
    for (int f = 0; f < FM; ++f) frag_off[f] = (wm * FM * 32 + f * 32) * ROWB + rd0;
#pragma unroll
    for (int f = 0; f < FN; ++f) frag_off[FM + f] = (BM + wn * FN * 32 + f * 32) * ROWB + rd0;
    auto read_frag = [&](int f, int stage, int ss) {
        return *reinterpret_cast<const u32x4 *>(smem + stage * STAGE + (frag_off[f] ^ (ss << 5)));
    };
    auto widen = [&](int f, const u32x4 &p) {
        v8i u;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            u[2 * w] = f < FM ? fp8_low(p[w]) : fp8_high(p[w]);
            u[2 * w + 1] = f < FM ? fp8_high(p[w]) : fp8_low(p[w]);
        }
        return u;
    };

    v16f acc[FM][FN];                                           // 2^-18 times the sums of the current group
    v16f facc[FM][FN];                                          // t1 + the zero-point sum

    // ---- first tile: requests for its first NS K steps and its token parameters ------------------------
    int vb = blockIdx.x;
    int tile = xcd_tile(vb, total);
    int m0 = (tile / g.tiles_n) * BM, n0 = (tile % g.tiles_n) * BN;
    __amdgpu_buffer_rsrc_t a_cur = a_desc(m0), b_cur = b_desc(n0);
    dma_tokens(m0, 0);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int i = 0; i < LD; ++i) dma_one(i, s, a_cur, b_cur, s * ROWB);
    __builtin_amdgcn_s_waitcnt(vmcnt_only((NS - 2) * LD));      // the first two K steps; the others are waited for at the barrier in front of each
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    // U: operands of the current sub-step, Un: of the next, P: codes of the one after it
    v8i U0[NF], U1[NF];
    u32x4 P[NF];

    int cur = 0;                                                // LDS stage of the current K step
    int parity = 0;
    for (;;) {
        // ---- tile start --------------------------------------------------------------------------------
        // (what the tile before has already read of this one is read again: the epilogue needs the registers)
#pragma unroll
        for (int f = 0; f < NF; ++f) P[f] = read_frag(f, cur, 0);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            U0[f] = widen(f, P[f]);
            P[f] = read_frag(f, cur, 1);
        }
        const int n_lane = n0 + wn * FN * 32 + (lane & 31) * FN;          // FN = 2 adjacent channels
        const int n_local = wn * FN * 32 + (lane & 31) * FN;
        const int vb_next = vb + stride;
        const bool has_next = vb_next < total;
        const int tile_next = xcd_tile(has_next ? vb_next : vb, total);
        const int m0n = (tile_next / g.tiles_n) * BM, n0n = (tile_next % g.tiles_n) * BN;
        const __amdgpu_buffer_rsrc_t a_nxt = a_desc(m0n, has_next), b_nxt = b_desc(n0n, has_next);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) facc[i][j][r] = 0.0f;

        // ---- main loop ---------------------------------------------------------------------------------
        // Weight scales of this lane's channels, four groups to a request (`held`: the last two, while the next request is under way),
        // and the zero-point tables' entries, zw of its channels and RA of its rows, of four groups too: lanes 0-31 the first two, lanes
        // 32-63 the others, which is how the fp32 MFMA wants them (two groups per instruction).  The last request of a row may reach past its
        // groups, into the next row, which is not used, or past the array, which reads as zeros: a descriptor's range check takes the
        // sum of vector and scalar offset, dword by dword.  (Ending with the row instead costs layers of few groups up to 8 %.)
        u32x4 quad[FN];
        float held[FN][2];
        u32x2 zw2[FN], ra2[FM];
        auto request_quad = [&](int grp0) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < FN; ++j) quad[j] = __builtin_amdgcn_raw_buffer_load_b128(sw_rsrc, (n_lane + j) * g.ng * 4, grp0 * 4, 0);
        };
        auto request_zero_points = [&](int grp0) __attribute__((always_inline)) {
            const int two = (lane >> 5) * 8;
#pragma unroll
            for (int j = 0; j < FN; ++j) zw2[j] = __builtin_amdgcn_raw_buffer_load_b64(zw_rsrc, (n_lane + j) * g.ng * 4 + two, grp0 * 4, 0);
#pragma unroll
            for (int i = 0; i < FM; ++i) ra2[i] = __builtin_amdgcn_raw_buffer_load_b64(ra_rsrc, (m0 + wm * FM * 32 + i * 32 + (lane & 31)) * g.ng * 4 + two, grp0 * 4, 0);
        };
        auto add_zero_points = [&](int k, int u) __attribute__((always_inline)) {
            facc[k / FN][k % FN] = __builtin_amdgcn_mfma_f32_32x32x2f32((float)(int)ra2[k / FN][u], __uint_as_float(zw2[k % FN][u]), facc[k / FN][k % FN], 0, 0, 0);
        };
        if constexpr (OUT != OUT_I32) request_quad(0);
        // t1 of fragment k += scale * sums of the group that is over
        auto fold = [&](int k, const float (&sc)[FN]) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 16; ++r) facc[k / FN][k % FN][r] = __fmaf_rn(sc[k % FN], acc[k / FN][k % FN][r], facc[k / FN][k % FN][r]);
        };
        // int32 export: the sums of group grp
        auto export_group = [&](int grp) __attribute__((always_inline)) {
            int32_t *plane = static_cast<int32_t *>(g.out) + (long)grp * g.M * g.N;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int m = m0 + wm * FM * 32 + frag_row(i, r, lane), n = n_lane + j;
                        if (m < g.M && n < g.N) plane[(long)m * g.N + n] = (int)(acc[i][j][r] * 262144.0f);
                    }
        };
        // One K step: SUB sub-steps of 64 codes.  In each the operands of the next are made of codes already in registers, and the
        // codes of the one after it are read.  Those of the next K step begin with the last sub-step but one: there its
        // stage has landed for every wave, and every wave has this stage's codes in registers, so that the barrier also frees this
        // stage for K step +NS.  Fragment k of the group before is folded in front of the MFMA that starts it anew, while the one before
        // runs.  kStart: the first step of a tile, with nothing to fold; 0 .. 3: place in a quad of groups; kTail: behind the last
        // quad.  Compile-time flags, and there is no branch in a step: the compiler would sink folds past it, and keep the sums
        // they wait for in memory.
        constexpr int kStart = -1, kTail = 4;
        auto k_step = [&](auto place_tag, int kt) __attribute__((always_inline)) {
            constexpr int Q = decltype(place_tag)::value;
            constexpr bool START = Q == kStart;
            const int nxt = cur == NS - 1 ? 0 : cur + 1;        // stage of stream step +1
            const bool own = kt + NS < KT;                      // stream step +NS is a step of this tile, or of the next one
            const __amdgpu_buffer_rsrc_t ra = own ? a_cur : a_nxt, rb = own ? b_cur : b_nxt;
            const int so = (own ? kt + NS : kt + NS - KT) * ROWB;
            float sc[FN];                                       // of the group to be folded
            if constexpr (!START && OUT != OUT_I32) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const float s = Q == 2 || Q == 3 ? held[j][Q & 1] : __uint_as_float(quad[j][Q == 1 ? 1 : 0]);
                    sc[j] = s * 262144.0f;
                    if constexpr (Q == 1) { held[j][0] = __uint_as_float(quad[j][2]); held[j][1] = __uint_as_float(quad[j][3]); }
                    if constexpr (Q == kTail) quad[j] = u32x4{quad[j][1], quad[j][2], quad[j][3], 0u};
                }
            }
#pragma unroll
            for (int ss = 0; ss < SUB; ++ss) {
                v8i (&Uc)[NF] = ss & 1 ? U1 : U0;
                v8i (&Un)[NF] = ss & 1 ? U0 : U1;
#pragma unroll
                for (int k = 0; k < NM; ++k) {
                    if (ss == 0) {
                        if constexpr (!START && OUT != OUT_I32) fold(k, sc);
                        __builtin_amdgcn_sched_barrier(0);      // (the accumulators may then be written in place)
                        const v16f zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                        acc[k / FN][k % FN] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(Uc[k / FN], Uc[FM + k % FN], zero, 0, 0, 0, 0, 0, 0);
                    } else {
                        acc[k / FN][k % FN] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(Uc[k / FN], Uc[FM + k % FN], acc[k / FN][k % FN], 0, 0, 0, 0, 0, 0);
                    }
                    if constexpr (Q == 3 && OUT != OUT_I32) add_zero_points(k, ss);
                    __builtin_amdgcn_sched_barrier(0);
                    if (ss == SUB - 2 && k == 0) {
                        // The next K step's requests are older than those of the NS - 2 steps behind it.  The first two steps of a tile have
                        // landed: a first tile begins with that, and later ones with all NS, waited for before the epilogue's stores.
                        if constexpr (START) __builtin_amdgcn_s_waitcnt(lds_only());
                        else __builtin_amdgcn_s_waitcnt(vmcnt_and_lds((NS - 2) * LD));
                        __builtin_amdgcn_s_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
                    }
                    if (k < NF) {
                        Un[k] = widen(k, P[k]);
                        P[k] = ss + 2 < SUB ? read_frag(k, cur, ss + 2) : read_frag(k, nxt, ss + 2 - SUB);
                    }
                    const int d = (ss - (SUB - 2)) * NM + k - (2 * NM - LD);   // tile DMAs in the last LD slots of the step
                    if (d >= 0) dma_one(d, cur, ra, rb, so);
                    if (ss == SUB - 1 && k == NM - 1) {
                        if constexpr (START) dma_tokens(m0n, parity ^ 1);
                        if constexpr (Q == 0 && OUT != OUT_I32) request_zero_points(kt - 1);
                        if constexpr (Q == 1 && OUT != OUT_I32) request_quad(kt + 2);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            cur = nxt;
        };
        k_step(std::integral_constant<int, kStart>{}, 0);
        if constexpr (OUT == OUT_I32) export_group(0);
        int kt = 1;
        if constexpr (OUT != OUT_I32) {
#pragma unroll
            for (int j = 0; j < FN; ++j) asm volatile("" : "+v"(quad[j]));     // waited for here, not (with all requests) in the loop
            do {                                                // (a tile has five groups at least: a way round the loop costs registers)
                k_step(std::integral_constant<int, 0>{}, kt);
                k_step(std::integral_constant<int, 1>{}, kt + 1);
                k_step(std::integral_constant<int, 2>{}, kt + 2);
                k_step(std::integral_constant<int, 3>{}, kt + 3);
                kt += 4;
            } while (kt + 4 <= KT);
            request_zero_points(kt - 1);                        // of the one to four groups that are left
        }
        const int rest = KT - (kt - 1);
        for (; kt < KT; ++kt) {
            k_step(std::integral_constant<int, kTail>{}, kt);
            if constexpr (OUT == OUT_I32) export_group(kt);
        }

        // ---- epilogue of this tile ------------------------------------------------------------------
        if constexpr (OUT != OUT_I32) {
            const u32x2 c_raw = __builtin_amdgcn_raw_buffer_load_b64(c_rsrc, n_lane * 4, 0, 0);
            const uint32_t bias_raw = __builtin_amdgcn_raw_buffer_load_b32(bias_rsrc, n_lane * 2, 0, 0);
            {
                float sc[FN];
#pragma unroll
                for (int j = 0; j < FN; ++j) sc[j] = __uint_as_float(quad[j][0]) * 262144.0f;
#pragma unroll
                for (int k = 0; k < NM; ++k) fold(k, sc);
            }
            constexpr int ESZ = OUT == OUT_F16 ? 2 : 4;
            const float *sa_lds = reinterpret_cast<const float *>(par + parity * (2 * BM * 4));
            const float *za_lds = sa_lds + BM;
            const __amdgpu_buffer_rsrc_t o_rsrc = make_rsrc(g.out, (uint32_t)((long)g.M * g.N * ESZ));
            const uint32_t row_bytes = (uint32_t)g.N * ESZ;
            const uint32_t col_off = n_lane < g.N ? (uint32_t)n_lane * ESZ : kPoison;
            const int row_w = wm * FM * 32;
            const uint32_t lane_off = (uint32_t)(m0 + row_w + 4 * (lane >> 5)) * row_bytes + col_off;
            const bool has_bias = g.bias != nullptr, gelu = g.act == W4A4_ACT_GELU;
            const float cv[FN] = {__uint_as_float(c_raw[0]), __uint_as_float(c_raw[1])};
            const float bv[FN] = {__half2float(__ushort_as_half((unsigned short)(bias_raw & 0xFFFFu))),
                                  __half2float(__ushort_as_half((unsigned short)(bias_raw >> 16)))};
            // the zero points of the groups behind the last quad; what lies past the last group belongs to another row
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const bool live = (lane >> 5) * 2 + u < rest;
#pragma unroll
                for (int i = 0; i < FM; ++i) ra2[i][u] = live ? ra2[i][u] : 0u;
#pragma unroll
                for (int j = 0; j < FN; ++j) zw2[j][u] = live ? zw2[j][u] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int k = 0; k < NM; ++k) add_zero_points(k, u);
            // every request of this tile and of the next one's first steps has landed: the next tile's first barriers need not wait
            // for the stores
            __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int rl = row_w + i * 32 + 8 * q + 4 * (lane >> 5);      // 4 consecutive rows
                    const float4 sa4 = *reinterpret_cast<const float4 *>(sa_lds + rl);
                    const float sav[4] = {sa4.x, sa4.y, sa4.z, sa4.w};
                    const float4 za4 = *reinterpret_cast<const float4 *>(za_lds + rl);
                    const float zav[4] = {za4.x, za4.y, za4.z, za4.w};
                    // y = fma(sa, t1 + sum_g zw*RA, fma(za, c, bias))
                    float y[4][FN];
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                        for (int j = 0; j < FN; ++j)
                            y[rr][j] = __fmaf_rn(sav[rr], facc[i][j][q * 4 + rr], __fmaf_rn(zav[rr], cv[j], has_bias ? bv[j] : 0.0f));
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const uint32_t off = lane_off + (uint32_t)(i * 32 + 8 * q + rr) * row_bytes;
                        if constexpr (OUT == OUT_F32) {
                            uint32_t w[FN];
#pragma unroll
                            for (int j = 0; j < FN; ++j) w[j] = __float_as_uint(gelu ? gelu_erf(y[rr][j]) : y[rr][j]);
                            store_words<FN, kStreamed>(o_rsrc, off, w);
                        } else if (gelu) {
                            store_gelu_halves<FN, kStreamed>(o_rsrc, off, y[rr]);
                        } else {
                            store_halves<FN, kStreamed>(o_rsrc, off, y[rr]);
                        }
                    }
                }
        } else {
            __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
        }
        if (!has_next) break;
        vb = vb_next; tile = tile_next; m0 = m0n; n0 = n0n; a_cur = a_nxt; b_cur = b_nxt; parity ^= 1;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));                  // no DMA may outlive the workgroup's LDS
}

template <int OUT>
static int launch_out(GemmArgs &g, hipStream_t st) {
    constexpr int BM = 128, BN = 128, NS = 4;
    constexpr size_t lds = NS * (BM + BN) * 64 + 2 * 2 * BM * 4;
    static_assert(lds <= kGroupLds, "two workgroups share a CU");
    if (g.steps_per_group != 1 || g.K / 128 < 5) return W4A4_ERR_UNSUPPORTED_SHAPE;
    g.tiles_m = (g.M + BM - 1) / BM;
    g.tiles_n = (g.N + BN - 1) / BN;
    auto kern = gemm_group_olay_kernel<OUT, NS>;
    static KernelState ks;
    const int cus = prepare_kernel(reinterpret_cast<const void *>(kern), lds, ks);
    if (cus < 0) return W4A4_ERR_HIP;
    const int slots = cus * 2;                                  // workgroups that are resident at once
    const long tiles = (long)g.tiles_m * g.tiles_n;
    if (tiles > 0x7fffffffL) return W4A4_ERR_UNSUPPORTED_SHAPE;
    const unsigned grid = (unsigned)(tiles < slots ? tiles : slots);
    launch_gemm(kern, dim3(grid), dim3(256), lds, st, g);
    return launch_status();
}

// Requires: asymmetric codes in the operand layout on both sides, weight groups of 128 codes; K % 128 == 0, K >= 640; M*lda, N*ldw, N*(ng+1)*4 and M*ng*4 < 2^31.
int launch_group_olay(int out_kind, GemmArgs &g, hipStream_t st) {
    switch (out_kind) {
        case OUT_F16: return launch_out<OUT_F16>(g, st);
        case OUT_F32: return launch_out<OUT_F32>(g, st);
        case OUT_I32: return launch_out<OUT_I32>(g, st);
        default: return W4A4_ERR_INVALID_ARG;
    }
}

}  // namespace w4a4
