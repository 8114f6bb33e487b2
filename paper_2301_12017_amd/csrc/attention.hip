// FP16 attention between the QKV projection and the attention output (Sec. 4.2 keeps the attention
// in FP16 and takes its kernel from elsewhere): softmax(q.k / sqrt(64)) V per sequence and head, no
// mask, on the FP16 matrix instruction with FP32 accumulation.
//
// A wave owns 32 queries and walks the keys in blocks of 32 with a running maximum.  It computes the
// scores TRANSPOSED (keys as rows: K Q^T), so that a lane holds sixteen scores of ONE query: the
// softmax needs a single exchange between the two halves of the wave, and the weights are already
// the B operand of the second product O^T = V^T P^T.  That product sums over keys in the order the
// first one leaves them in (eight per half: 0..3 and 8..11, or 4..7 and 12..15 of every sixteen); V
// is read from LDS in the same order with the transposing load.
//
// A weight is the sum of two FP16 numbers, p = hi + lo (the matrix instruction takes subnormal ones), so the second
// product costs two matrix instructions per operand of V.  They hold 2^15 p, p <= 1: 22 bits down to weights of 2^-29, and
// no worse than 2^-41 below, where p itself would lose 2^-26.  Weights of e^-18 keep the digits that an FP16 result can show,
// as it does where the largest weight meets a value of zero.
//
// Bound by the vector ALU between the products (per score: exponent, v_exp at a quarter of the rate, sum, split into two
// halves), not by memory: 24 x 512 tokens, 16 heads: 54 us, where the kernel it replaced (one query at a time per wave, v_dot2
// scores and an FMA per key and feature) took 1765 us and the bytes 19 us; 128 x 128 tokens, 12 heads: 22 us (274 us);
// 1 x 128: 3.9 us (6.1 us), 1 x 32: 3.2 us (3.5 us), near the launch floor.
#include "common.hpp"

namespace w4a4 {
namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short short4_t __attribute__((__vector_size__(8)));
typedef __attribute__((address_space(3))) short4_t lds_short4;

constexpr int kHead = 64;             // features per head
constexpr int kAttnThreads = 256;
constexpr int kRowHalves = 72;        // LDS pitch of a key / value row: 144 bytes, rows start in different banks
constexpr float kScoreScale = 0.125f * 1.44269504f;   // 1 / sqrt(64), base 2
constexpr float kWeightScale = 32768.0f;              // of the largest weight, 1, where weights are split in two halves

__device__ __forceinline__ uint32_t pack_halves(float a, float b) {      // round to nearest even
    const float2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, half2_t));
}

// Two weights as two pairs of halves: p = hi + lo.  (v_fma_mixlo / mixhi would round both halves in two instructions each and need
// no multiply, but are slower: 24 x 512 tokens 55 us, 53 so.)
__device__ __forceinline__ void split(float p0, float p1, uint32_t &hi, uint32_t &lo) {
    hi = pack_halves(p0, p1);
    float r0, r1;                     // p - hi, exact
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(hi), "v"(p0));
    asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(hi), "v"(p1));
    lo = pack_halves(r0, r1);
}

// op over the two lanes l, l + 32 of a wave, in both of them
template <typename Op>
__device__ __forceinline__ float both_halves(float x, Op op) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    return op(__builtin_bit_cast(float, (unsigned)sw[0]), __builtin_bit_cast(float, (unsigned)sw[1]));
}

// The weight of a key with raw score s is exp2(s * kScoreScale + shift), one FMA, in a row whose largest raw score is m.  The
// shift is a rounded number, but the same one for every weight and for the sum of them, so that its rounding cancels.  That
// ends where it moves the largest weight itself (a quarter of a power of two at 2^22, 32 of them at 2^29): there, and for
// infinite m, the scores are taken relative to m first (`far`).
__device__ __forceinline__ float weight_shift(float m) { return -m * kScoreScale; }
__device__ __forceinline__ bool far(float shift) { return !(fabsf(shift) < 4194304.0f); }
// what turns weights of a row with maximum m0 into those of maximum m (nothing has been summed yet while m0 is -inf)
__device__ __forceinline__ float weight_ratio(float m0, float m) {
    const float s0 = weight_shift(m0), s = weight_shift(m);
    const float e = far(s0) || far(s) ? (m0 - m) * kScoreScale : s - s0;
    return m0 > -INFINITY ? __builtin_amdgcn_exp2f(e) : 0.0f;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const _Float16 *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16 *>(p), (short)0, (int)bytes, 0x00020000);
}

// State of a wave's 32 queries: lane l belongs to query l % 32 and holds features 32 f + 8 (i / 4) + 4 (l / 32) + i % 4.
struct QueryBlock {
    half8_t q[4];                     // B operands: features 16 s + 8 (l / 32) ..+7 of the lane's query
    float16_t o[2];
    float m, l;                       // running maximum of the raw scores; the lane's half of the sum
    float shift, settled;             // of its weights; maximum of a block up to which neither changes (far rows: none)
};

// One block of 32 keys: rows 0..31 of the LDS tiles ks / vs, of which the first `valid` are keys.
__device__ __forceinline__ void attend32(QueryBlock &Q, const _Float16 *ks, const _Float16 *vs, int lane, int valid) {
    const int row = lane & 31, hl = lane >> 5;
    float16_t s = {};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const half8_t k = *reinterpret_cast<const half8_t *>(ks + row * kRowHalves + 16 * t + 8 * hl);
        s = __builtin_amdgcn_mfma_f32_32x32x16_f16(k, Q.q[t], s, 0, 0, 0);
    }
    if (valid < 32) {                 // wave-uniform: the last block of a sequence
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (8 * (i / 4) + i % 4 >= valid - 4 * hl) s[i] = -INFINITY;
    }
    // (v_max3_f32, but by the compiler: it does not see what inline assembly reads and would leave out the wait states that
    // a read of a matrix instruction's result needs)
    float mx = Q.m;
#pragma unroll
    for (int i = 0; i < 16; i += 2) mx = fmaxf(fmaxf(mx, s[i]), s[i + 1]);
    mx = both_halves(mx, [](float x, float y) { return fmaxf(x, y); });
    if (__any(mx > Q.settled)) {      // wave-uniform, seldom taken after the first blocks
        const float a = weight_ratio(Q.m, mx);
        Q.m = Q.settled = mx;
        Q.shift = mx > -INFINITY ? weight_shift(mx) : 0.0f;        // (keys of score -inf alone: weights 0)
        Q.l *= a;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int i = 0; i < 16; ++i) Q.o[f][i] *= a;
        if (__builtin_expect(__any(far(Q.shift)), 0) && far(Q.shift)) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] -= mx;
            Q.shift = weight_shift(0.0f);
            Q.settled = -INFINITY;
        }
    }
    uint32_t hi[8], lo[8];
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * i], kScoreScale, Q.shift));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * i + 1], kScoreScale, Q.shift));
        sum += p0 + p1;
        split(p0 * kWeightScale, p1 * kWeightScale, hi[i], lo[i]);
    }
    Q.l += sum;
    // the lane's address in a transposing load: row (lane % 16) / 4 of four, columns 4 (lane % 4) of sixteen
    const _Float16 *vrow = vs + (4 * hl + ((lane & 15) >> 2)) * kRowHalves + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        struct B2 { uint32_t w[4]; };
        const half8_t ph = __builtin_bit_cast(half8_t, (B2{{hi[4 * t], hi[4 * t + 1], hi[4 * t + 2], hi[4 * t + 3]}}));
        const half8_t pl = __builtin_bit_cast(half8_t, (B2{{lo[4 * t], lo[4 * t + 1], lo[4 * t + 2], lo[4 * t + 3]}}));
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            struct S2 { short4_t a, b; } v;
            v.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(vrow + (16 * t) * kRowHalves + 32 * f));
            v.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(vrow + (16 * t + 8) * kRowHalves + 32 * f));
            const half8_t vf = __builtin_bit_cast(half8_t, v);
            Q.o[f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, ph, Q.o[f], 0, 0, 0);
            Q.o[f] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf, pl, Q.o[f], 0, 0, 0);
        }
    }
}

// Results that hold a NaN although the row's sum of weights does not: a value among V is infinite or NaN, and a split weight
// gives NaN where the definition need not (a half of it is negative or zero).  What the definition has in such a feature is
// decided by those values alone: the sum of weight * value over them, with the weights in FP32.  Each key that has one among the
// sixteen features 8 blk .. 8 blk + 15 of the wave's two halves is scored again, by the whole wave.  16 x 512 tokens, 12 heads,
// 33 us: 37 us with a NaN, 39 us with an infinity among each head's values, 1.1 ms with nothing but infinities.
__device__ void special_values(const _Float16 *base, long ld, int h, int seq, int lane, const half8_t (&q)[4], float m, float l, int blk,
                               float (&x)[4], float (&y)[4]) {
    const int hl = lane >> 5;
    const _Float16 *k = base + h, *v = base + 2 * h + 8 * blk;
    float sx[4] = {}, sy[4] = {};
    auto special = [](_Float16 f) { return (__builtin_bit_cast(unsigned short, f) & 0x7C00) == 0x7C00; };
#pragma unroll 1
    for (int k0 = 0; k0 < seq; k0 += kWave) {
        bool found = false;
        if (k0 + lane < seq) {
            const half8_t a = *reinterpret_cast<const half8_t *>(v + (k0 + lane) * ld), b = *reinterpret_cast<const half8_t *>(v + (k0 + lane) * ld + 8);
#pragma unroll
            for (int i = 0; i < 8; ++i) found |= special(a[i]) || special(b[i]);
        }
#pragma unroll 1
        for (unsigned long long todo = __ballot(found); todo; todo &= todo - 1) {
            const int key = k0 + __builtin_ctzll(todo);
            float s = 0.0f;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const half8_t kt = *reinterpret_cast<const half8_t *>(k + key * ld + 16 * t + 8 * hl);
#pragma unroll
                for (int i = 0; i < 8; i += 2) s = __builtin_amdgcn_fdot2(half2_t{q[t][i], q[t][i + 1]}, half2_t{kt[i], kt[i + 1]}, s, false);
            }
            const float p = expf((both_halves(s, [](float x, float y) { return x + y; }) - m) * 0.125f);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const _Float16 vx = v[key * ld + 4 * hl + i], vy = v[key * ld + 8 + 4 * hl + i];
                if (special(vx)) sx[i] = __builtin_fmaf(p, (float)vx, sx[i]);
                if (special(vy)) sy[i] = __builtin_fmaf(p, (float)vy, sy[i]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (l > 0.0f && sx[i] != 0.0f) x[i] = sx[i];
        if (l > 0.0f && sy[i] != 0.0f) y[i] = sy[i];
    }
}

// One workgroup of four waves per block of queries of one (sequence, head).  SPLIT == 1: a wave per 32 queries, 128
// queries, keys and values staged 64 rows at a time and shared by the four.  SPLIT == 4: 32 queries, the waves take a
// quarter of every 128 staged keys each and add up their parts through LDS: for launches that would leave CUs idle.
template <int SPLIT>
__global__ __launch_bounds__(kAttnThreads, SPLIT == 1 ? 4 : 3) void attention_mfma_kernel(const __half *qkv, __half *ctx, int seq, int heads,
                                                                      int pairs, int qblocks) {
    constexpr int TILE = SPLIT == 4 ? 128 : 64, CH = TILE / 32;
    extern __shared__ __attribute__((aligned(16))) _Float16 smem[];           // [buffers][keys, values][TILE][kRowHalves]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hl = lane >> 5;
    // the query blocks of a (sequence, head) run on one XCD: they share its keys and values in that L2
    const int loc = blockIdx.x >> 3, pair = (loc / qblocks) * 8 + (blockIdx.x & 7), qb = loc % qblocks;
    if (pair >= pairs) return;
    const int b = pair / heads, head = pair % heads, h = heads * kHead;
    const long ld = 3L * h;
    const _Float16 *base = reinterpret_cast<const _Float16 *>(qkv) + (long)b * seq * ld + head * kHead;
    const int q0 = SPLIT == 4 ? qb * 32 : qb * 128 + wave * 32;
    const int qi = q0 + (lane & 31);

    // 32-bit offsets from uniform bases; for SPLIT == 1 through descriptors that end with the sequence, for SPLIT == 4 under a
    // condition (rows behind the sequence are zero in both).  Descriptors | conditions | 64-bit addresses, us: 24 x 512 tokens
    // 53.6 | 54.2 | 55.4, 9 x 371 16.1 | 16.6 | 16.7, 1 x 32 3.17 | 3.22 | 3.27; with keys split over the waves, 1 x 128,
    // descriptors cost 0.1.
    u32x4 kreg[CH], vreg[CH];
    const int srow = tid >> 3, scol = (tid & 7) * 8;
    const uint32_t ld_bytes = (uint32_t)ld * 2, bytes = (uint32_t)(seq - 1) * ld_bytes + kHead * 2, off0 = srow * ld_bytes + scol * 2;
    const __amdgpu_buffer_rsrc_t k_rsrc = rows_rsrc(base + h, bytes), v_rsrc = rows_rsrc(base + 2 * h, bytes);
    auto fetch = [&](int tile) {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int r = tile * TILE + 32 * j;
            if constexpr (SPLIT == 1) {
                kreg[j] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, off0 + r * ld_bytes, 0, 0);
                vreg[j] = __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, off0 + r * ld_bytes, 0, 0);
            } else {
                const char *kb = reinterpret_cast<const char *>(base + h), *vb = reinterpret_cast<const char *>(base + 2 * h);
                kreg[j] = vreg[j] = u32x4{0, 0, 0, 0};
                if (r + srow < seq) {
                    kreg[j] = *reinterpret_cast<const u32x4 *>(kb + (off0 + r * ld_bytes));
                    vreg[j] = *reinterpret_cast<const u32x4 *>(vb + (off0 + r * ld_bytes));
                }
            }
        }
    };
    auto put = [&](int buf) {
        _Float16 *d = smem + buf * 2 * TILE * kRowHalves + srow * kRowHalves + scol;
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            *reinterpret_cast<u32x4 *>(d + 32 * j * kRowHalves) = kreg[j];
            *reinterpret_cast<u32x4 *>(d + (TILE + 32 * j) * kRowHalves) = vreg[j];
        }
    };

    QueryBlock Q;
    fetch(0);
    {
        const _Float16 *qp = base + (qi < seq ? qi : seq - 1) * ld + 8 * hl;
#pragma unroll
        for (int t = 0; t < 4; ++t) Q.q[t] = *reinterpret_cast<const half8_t *>(qp + 16 * t);
    }
    Q.o[0] = float16_t{};
    Q.o[1] = float16_t{};
    Q.m = -INFINITY;
    Q.settled = -INFINITY;
    Q.l = Q.shift = 0.0f;
    put(0);
    const int tiles = (seq + TILE - 1) / TILE;
    if (tiles > 1) fetch(1);
    __syncthreads();
    for (int t = 0; t < tiles; ++t) {
        const _Float16 *ks = smem + (t & 1) * 2 * TILE * kRowHalves, *vs = ks + TILE * kRowHalves;
        if (SPLIT == 4) {
            const int left = seq - t * TILE - wave * 32;
            if (left > 0) attend32(Q, ks + wave * 32 * kRowHalves, vs + wave * 32 * kRowHalves, lane, left);
        } else if (q0 < seq) {
            attend32(Q, ks, vs, lane, seq - t * TILE);
            if (t * TILE + 32 < seq) attend32(Q, ks + 32 * kRowHalves, vs + 32 * kRowHalves, lane, seq - t * TILE - 32);
        }
        if (t + 1 < tiles) {
            put((t + 1) & 1);
            if (t + 2 < tiles) fetch(t + 2);
            __syncthreads();
        }
    }

    __half *dst = ctx + ((long)b * seq + qi) * h + head * kHead;
    float l = both_halves(Q.l, [](float x, float y) { return x + y; });
    // Two blocks of four features of a lane and of its partner in the other half make eight consecutive ones each:
    // features 8 blk..+7 for the lower half, 8 (blk + 1)..+7 for the upper one, sixteen bytes per lane.
    auto store16 = [&](float (&x)[4], float (&y)[4], float l, float m, int blk) {
        const float any = ((x[0] + x[1]) + (x[2] + x[3])) + ((y[0] + y[1]) + (y[2] + y[3]));
        // (a sum of weights that is NaN or 0 means a NaN in the definition: a score that is NaN or +inf, or only -inf ones)
        if (__builtin_expect(__any(any != any && l > 0.0f), 0)) special_values(base, ld, h, seq, lane, Q.q, m, l, blk, x, y);
        const uint32_t x0 = pack_halves(x[0], x[1]), x1 = pack_halves(x[2], x[3]);
        const uint32_t y0 = pack_halves(y[0], y[1]), y1 = pack_halves(y[2], y[3]);
        const auto s0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
        if (qi < seq) *reinterpret_cast<uint4 *>(dst + 8 * (blk + hl)) = uint4{(uint32_t)s0[0], (uint32_t)s1[0], (uint32_t)s0[1], (uint32_t)s1[1]};
    };
    if (SPLIT == 1) {
        if (q0 >= seq) return;
        const float inv = 1.0f / (l * kWeightScale);
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int g = 0; g < 4; g += 2) {
                float x[4], y[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { x[i] = Q.o[f][4 * g + i] * inv; y[i] = Q.o[f][4 * g + 4 + i] * inv; }
                store16(x, y, l, Q.m, 4 * f + g);
            }
        return;
    }
    // the four waves' parts of the same queries: maxima first, then the rescaled sums and outputs
    float *part = reinterpret_cast<float *>(smem);                            // [4 waves][32 registers][64 lanes]
    float *ml = part + 4 * 32 * 64;                                           // [4 waves][32 queries]: maxima, then sums
    __syncthreads();
    if (hl == 0) ml[wave * 32 + lane] = Q.m;
    __syncthreads();
    float m = ml[lane & 31];
#pragma unroll
    for (int w = 1; w < 4; ++w) m = fmaxf(m, ml[w * 32 + (lane & 31)]);
    const float a = weight_ratio(Q.m, m);                                     // 0 for a wave without keys
    if (hl == 0) ml[128 + wave * 32 + lane] = l * a;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int i = 0; i < 16; ++i) part[(wave * 32 + 16 * f + i) * 64 + lane] = Q.o[f][i] * a;
    __syncthreads();
    l = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) l += ml[128 + w * 32 + (lane & 31)];
    const float inv = 1.0f / (l * kWeightScale);
    float x[4], y[4];                                                         // wave w finishes registers 8 w .. 8 w + 7
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float u = 0.0f, v = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            u += part[(w * 32 + 8 * wave + i) * 64 + lane];
            v += part[(w * 32 + 8 * wave + 4 + i) * 64 + lane];
        }
        x[i] = u * inv;
        y[i] = v * inv;
    }
    store16(x, y, l, m, 2 * wave);
}

constexpr size_t tile_bytes(int tile) { return (size_t)2 * tile * kRowHalves * sizeof(_Float16); }

template <int SPLIT>
int launch_attention(const void *qkv, void *ctx, int batch, int seq, int heads, hipStream_t st) {
    constexpr int TILE = SPLIT == 4 ? 128 : 64, QB = SPLIT == 4 ? 32 : 128;
    const int pairs = batch * heads, qblocks = (seq + QB - 1) / QB;
    size_t lds = tile_bytes(TILE) * (seq > TILE ? 2 : 1);
    const size_t combine = (size_t)(4 * 32 * 64 + 256) * sizeof(float);
    if (SPLIT == 4 && lds < combine) lds = combine;
    static KernelState ks;
    if (prepare_kernel(reinterpret_cast<const void *>(attention_mfma_kernel<SPLIT>), lds, ks) < 0) return W4A4_ERR_HIP;
    hipLaunchKernelGGL((attention_mfma_kernel<SPLIT>), dim3((unsigned)((pairs + 7) / 8 * 8 * qblocks)), dim3(kAttnThreads), lds, st,
                       static_cast<const __half *>(qkv), static_cast<__half *>(ctx), seq, heads, pairs, qblocks);
    return launch_status();
}

}  // namespace
}  // namespace w4a4

using namespace w4a4;

extern "C" int w4a4_attention_f16(const void *QKV_f16, int batch, int seq, int heads, void *ctx_f16, void *stream) {
    if (batch < 0 || seq < 0 || heads <= 0) return W4A4_ERR_INVALID_ARG;
    if (batch == 0 || seq == 0) return W4A4_OK;
    if (!QKV_f16 || !ctx_f16) return W4A4_ERR_INVALID_ARG;
    if (seq > 512 || heads > 1024) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if (!aligned16(QKV_f16) || !aligned16(ctx_f16)) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if ((long)batch * seq * 3 * heads * kHead >= 0x7fffffffL) return W4A4_ERR_UNSUPPORTED_SHAPE;
    // 128 queries per workgroup share each staged tile; below 192 such workgroups most CUs idle and 32 queries per
    // workgroup, keys split over its waves, are faster.  us at 128 | 32 queries, twelve heads: 1 x 128 tokens (12 workgroups
    // of 128) 5.5 | 3.9, 5 x 93 (60) 5.1 | 4.1, 16 x 128 (192) 6.3 | 6.9, 4 x 512 (192) 16.1 | 15.1, 64 x 128 (768) 13.9 | 19.3.
    // With one block of keys there is nothing to split, and the combination of the waves' parts is left out: 1 x 8 tokens
    // 3.3 | 3.8, 1 x 32 3.2 | 3.7, 15 x 32 3.3 | 3.8; with two, 1 x 33 4.0 | 3.9, 1 x 64 3.9 | 3.8.
    if (seq <= 32 || (long)batch * heads * ((seq + 127) / 128) >= 192)
        return launch_attention<1>(QKV_f16, ctx_f16, batch, seq, heads, as_stream(stream));
    return launch_attention<4>(QKV_f16, ctx_f16, batch, seq, heads, as_stream(stream));
}
