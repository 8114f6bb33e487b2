// Per-part quantization strategy (Sec. 4.2, last paragraphs; Sec. 4.3): the four linear parts of
// an encoder layer as components that run in INT4 or in the INT8 sibling, the FFN pair with or
// without the codes handed over in FFN1's epilogue, and the tuner that measures every option on
// the device it runs on and picks the cheapest combination.  Host code over the library's own
// entry points; the only kernels here fill the tuner's synthetic operands.
#include <math.h>

#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "layer.hpp"

namespace w4a4 {
namespace {

constexpr size_t kAlign = 256;
inline size_t up(size_t b) { return (b + kAlign - 1) / kAlign * kAlign; }

// Carves 256-byte aligned pieces off a workspace; `need` only adds up when base is null.
struct Carver {
    uint8_t *base;
    size_t used = 0;
    explicit Carver(void *b) : base(static_cast<uint8_t *>(b)) {}
    template <typename T>
    T *take(size_t count) {
        T *p = base ? reinterpret_cast<T *>(base + used) : nullptr;
        used += up(count * sizeof(T));
        return p;
    }
};

int groups_of(const w4a4_weight &w) { return (w.group == 0 || w.group >= w.K) ? 1 : w.K / w.group; }

// Buffers of a token-wise quantized activation matrix [M, K] that matches weights `w`.
struct ActBuffers {
    uint8_t *q; float *scale, *zero; int32_t *gsum, *osum;
};
// bytes of its codes: two per byte, or - FP6 operand layout - whole 64-token panels of 3/4 byte per code
size_t act_code_bytes(int M, int K, int layout) {
    return layout == W4A4_LAYOUT_FP6 ? (((size_t)M + 63) & ~(size_t)63) * (K / 4 * 3) : (size_t)M * (K / 2);
}
ActBuffers carve_act4(Carver &c, int M, int K, const w4a4_weight &w) {
    ActBuffers b;
    b.q = c.take<uint8_t>(act_code_bytes(M, K, w.layout));
    b.scale = c.take<float>(M);
    b.zero = c.take<float>(M);
    b.gsum = c.take<int32_t>((size_t)M * groups_of(w));
    b.osum = c.take<int32_t>((size_t)M * groups_of(w));         // one word per token (symmetric) or per token and group
    return b;
}
w4a4_act view_act4(const ActBuffers &b, int M, int K, const w4a4_weight &w) {
    w4a4_act a;
    a.q = b.q; a.scale = b.scale;
    a.zero = w.mode == W4A4_ASYM ? b.zero : nullptr;
    a.gsum = w.mode == W4A4_ASYM ? b.gsum : nullptr;
    a.M = M; a.K = K; a.lda = w.layout == W4A4_LAYOUT_FP6 ? K / 4 * 3 : K / 2; a.group = w.group; a.mode = w.mode; a.layout = w.layout;
    a.osum = w.layout == W4A4_LAYOUT_MFMA ? b.osum : nullptr;
    a.ldo = 1;
    return a;
}

size_t part_bytes(int M, const w4a4_part &p) {
    const int K = p.w4.K;
    Carver c4(nullptr);
    carve_act4(c4, M, K, p.w4);
    Carver c8(nullptr);
    c8.take<int8_t>((size_t)M * K);
    c8.take<float>(M);
    return c4.used > c8.used ? c4.used : c8.used;
}

bool part_ok(const w4a4_part *p) {
    return p && p->w4.N > 0 && p->w4.K > 0 && p->w4.K % 32 == 0 && (p->act == W4A4_ACT_NONE || p->act == W4A4_ACT_GELU);
}

// One launch for small token counts, whose workgroups quantize their tokens' whole rows.  INT4: up to 960 tiles of 32 x 32 (us, one launch |
// two: 300 x 3072 x 768 (960) 6.0 | 6.3, 465 x 2304 x 768 (1080) 7.9 | 7.6, 300 x 3072 x 1024 (960) 6.95 | 6.85, 224 x 4096 x 1024 (896) 6.9 | 6.9, 384 x 3072 x 1024
// (1152) 9.2 | 8.3), 512 of K > 1024; with long rows only up to 128, where the kernel still takes tiles of 8 or 16 tokens: 160 x 768 x 3072 (120) 5.3 | 6.2,
// 224 x 768 x 3072 (168) 7.2 | 6.6.  Where the kernel has K at run time, which costs it some 30 %, more than 512 tiles take one launch up to 600 tokens:
// 507 x 1920 x 640 (960) 6.9 | 7.2, 411 x 2304 x 576 (936) 6.9 | 7.1, 923 x 640 x 640 (580) 7.1 | 7.15, 1179 x 640 x 640 (740) 8.1 | 7.3, 1691 x 576 x 576 (954) 8.5 | 7.2,
// 603 x 960 x 960 (570) 8.9 | 8.8, 1019 x 960 x 960 (960) 9.3 | 8.9.  INT8: 512; 465 x 768 x 3072 12.8 | 14.5.
bool one_kernel_tiles(int M, int N, int K, bool int4) {
    const long tiles = (long)((M + 31) / 32) * ((N + 31) / 32);
    return K % 64 == 0 && K <= 4096 && tiles <= (!int4 ? 512 : K > 2048 ? 128 : K > 1024 || (!small_constant_k(K) && M > 600) ? 512 : 960);
}
// ... symmetric per-channel weights in the canonical layout
bool one_kernel_shape(int M, const w4a4_weight &w) {
    return w.layout == W4A4_LAYOUT_CANONICAL && w.mode == W4A4_SYM && groups_of(w) == 1 && one_kernel_tiles(M, w.N, w.K, true);
}
// FFN1 of a layer: there the alternative is not a launch more, since LayerNorm's kernel writes the codes, and the one launch forms
// LayerNorm for every column tile: up to 512 tiles (layer of 768 at 1 x 128 tokens, 384 tiles, 27.8 us in one | 28.4; 2 x 128, 768 tiles, 37.5 | 33.2).
bool one_kernel_ffn1(int M, const w4a4_weight &w) {
    return one_kernel_shape(M, w) && (long)((M + 31) / 32) * ((w.N + 31) / 32) <= 512;
}

int run_part(const void *X, int M, int ldx, const w4a4_part &p, bool int4, void *out, void *ws, void *stream) {
    const int K = p.w4.K, N = p.w4.N;
    w4a4_epilogue ep = {};
    ep.bias_f16 = p.bias_f16;
    ep.act = p.act;
    if (int4) {
        if (one_kernel_shape(M, p.w4)) {
            const int rc = w4a4_linear_f16act(X, M, K, ldx, &p.w4, &ep, out, stream);
            if (rc != W4A4_ERR_UNSUPPORTED_SHAPE) return rc;
        }
        Carver c(ws);
        const ActBuffers b = carve_act4(c, M, K, p.w4);
        const w4a4_act a = view_act4(b, M, K, p.w4);
        int rc = w4a4_quantize_act(X, M, K, ldx, p.w4.mode, p.w4.group, b.q, b.scale, a.zero ? b.zero : nullptr,
                                   a.gsum ? b.gsum : nullptr, p.w4.layout, b.osum, stream);
        if (rc) return rc;
        return w4a4_linear(&a, &p.w4, &ep, out, nullptr, nullptr, nullptr, nullptr, 0, stream);
    }
    if (!p.w8q || !p.w8s) return W4A4_ERR_INVALID_ARG;
    if (one_kernel_tiles(M, N, K, false)) {
        const int rc = w8a8_linear_f16act(X, M, K, ldx, p.w8q, p.w8s, N, &ep, out, stream);
        if (rc != W4A4_ERR_UNSUPPORTED_SHAPE) return rc;
    }
    Carver c(ws);
    int8_t *q = c.take<int8_t>((size_t)M * K);
    float *s = c.take<float>(M);
    int rc = w8a8_quantize_rows(X, M, K, ldx, q, s, stream);
    if (rc) return rc;
    return w8a8_linear(q, K, s, M, p.w8q, p.w8s, N, K, &ep, out, stream);
}

// ---- FFN pair -----------------------------------------------------------------------------------
struct FusedPlan {
    ActBuffers a1, h;
    void *lin_ws;
    size_t lin_bytes;
    size_t total;
};
w4a4_epilogue fused_epilogue(const w4a4_part &f1, const w4a4_part &f2) {
    w4a4_epilogue ep = {};
    ep.bias_f16 = f1.bias_f16;
    ep.act = f1.act;
    ep.requant = 1;
    ep.requant_mode = W4A4_SYM;
    ep.requant_group = 0;
    ep.requant_layout = f2.w4.layout;
    return ep;
}
FusedPlan plan_fused(void *ws, int M, const w4a4_part &f1, const w4a4_part &f2) {
    Carver c(ws);
    FusedPlan p;
    p.a1 = carve_act4(c, M, f1.w4.K, f1.w4);
    p.h = carve_act4(c, M, f2.w4.K, f2.w4);
    const w4a4_act a1 = view_act4(p.a1, M, f1.w4.K, f1.w4);
    const w4a4_epilogue ep = fused_epilogue(f1, f2);
    p.lin_bytes = w4a4_linear_workspace_bytes(&a1, &f1.w4, &ep, f2.w4.layout == W4A4_LAYOUT_MFMA);
    p.lin_ws = c.take<uint8_t>(p.lin_bytes);
    p.total = c.used;
    return p;
}
size_t unfused_bytes(int M, const w4a4_part &f1, const w4a4_part &f2) {
    const size_t a = part_bytes(M, f1), b = part_bytes(M, f2);
    return up((size_t)M * f1.w4.N * 2) + (a > b ? a : b);
}

// ---- whole encoder layer ------------------------------------------------------------------------
struct LayerPlan {
    __half *qkv, *ctx, *ao, *x1, *h2;
    ActBuffers ln;                  // codes of LayerNorm 1 for FFN1
    uint8_t *rest;                  // whatever the part that is running needs
    size_t rest_bytes, total;
};
bool layer_ok(const w4a4_encoder_layer_weights *L) {
    if (!L || L->hidden <= 0 || L->heads <= 0 || L->ffn <= 0 || L->hidden != L->heads * 64) return false;
    if (!part_ok(&L->qkv) || !part_ok(&L->attn_out) || !part_ok(&L->ffn1) || !part_ok(&L->ffn2)) return false;
    const int h = L->hidden, f = L->ffn;
    return L->qkv.w4.N == 3 * h && L->qkv.w4.K == h && L->attn_out.w4.N == h && L->attn_out.w4.K == h &&
           L->ffn1.w4.N == f && L->ffn1.w4.K == h && L->ffn2.w4.N == h && L->ffn2.w4.K == f &&
           L->ffn1.w4.mode == W4A4_SYM && L->ffn2.w4.mode == W4A4_SYM && groups_of(L->ffn1.w4) == 1 &&
           L->ln1_gamma_f16 && L->ln1_beta_f16 && L->ln2_gamma_f16 && L->ln2_beta_f16 && L->ln_eps >= 0.0f;
}
LayerPlan plan_layer(void *ws, int M, const w4a4_encoder_layer_weights &L) {
    Carver c(ws);
    LayerPlan p;
    const size_t h = L.hidden;
    p.qkv = c.take<__half>((size_t)M * 3 * h);
    p.ctx = c.take<__half>((size_t)M * h);
    p.ao = c.take<__half>((size_t)M * h);
    p.x1 = c.take<__half>((size_t)M * h);
    p.h2 = c.take<__half>((size_t)M * h);
    p.ln = carve_act4(c, M, L.hidden, L.ffn1.w4);
    size_t r = w4a4_ffn_workspace_bytes(M, &L.ffn1, &L.ffn2);   // covers both ways FFN1 can take LayerNorm's codes, too
    const size_t a = part_bytes(M, L.qkv), b = part_bytes(M, L.attn_out);
    r = r > a ? r : a;
    r = r > b ? r : b;
    p.rest_bytes = r;
    p.rest = c.take<uint8_t>(r);
    p.total = c.used;
    return p;
}

LnArgs layernorm_args(const void *X, const void *R, int M, int K, const void *gamma, const void *beta, float eps, void *Y) {
    LnArgs a = {};
    a.X = static_cast<const __half *>(X); a.R = static_cast<const __half *>(R); a.ldx = K;
    a.gamma = static_cast<const __half *>(gamma); a.beta = static_cast<const __half *>(beta);
    a.eps = eps; a.Y = static_cast<__half *>(Y);
    a.M = M; a.K = K;
    return a;
}

// y (and codes of it, if asked for) = LayerNorm(X + R): the kernel of w4a4_layernorm_quantize, symmetric codes in `layout`
int run_layernorm(const void *X, const void *R, int M, int K, const void *gamma, const void *beta, float eps, void *Y,
                  const ActBuffers &b, int layout, int codes, const ClearRanges &clear, void *stream) {
    int lpr = 0, opl = 0;
    if (K % 32 || K > 4096 || (codes != LN_CODES_NONE && layout == W4A4_LAYOUT_FP6 && !fp6_plan(K, &lpr, &opl))) return W4A4_ERR_UNSUPPORTED_SHAPE;
    for (const void *p : {X, R, gamma, beta, static_cast<const void *>(Y)})
        if (!aligned16(p)) return W4A4_ERR_UNSUPPORTED_SHAPE;
    LnArgs a = layernorm_args(X, R, M, K, gamma, beta, eps, Y);
    a.q = b.q; a.s = b.scale; a.z = nullptr; a.gsum = nullptr; a.ng = 1; a.cpg = K / 8; a.psum = b.osum;
    a.zero0 = clear.p0; a.n0 = clear.n0; a.zero1 = clear.p1; a.n1 = clear.n1;
    return layernorm_rows(a, layout, codes, as_stream(stream));
}

// ---- tuner --------------------------------------------------------------------------------------
__global__ void fill_bytes_kernel(uint32_t *p, size_t words, uint32_t seed) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x) {
        uint32_t x = (uint32_t)i * 0x9E3779B9u + seed;          // an integer hash: every byte looks random
        x ^= x >> 16; x *= 0x7FEB352Du; x ^= x >> 15; x *= 0x846CA68Bu; x ^= x >> 16;
        p[i] = x;
    }
}
__global__ void fill_halves_kernel(__half *p, size_t n, uint32_t seed, float amp) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        uint32_t x = (uint32_t)i * 0x9E3779B9u + seed;
        x ^= x >> 16; x *= 0x7FEB352Du; x ^= x >> 15; x *= 0x846CA68Bu; x ^= x >> 16;
        // the sum of two uniforms: a bell-ish spread, so that a token uses most of the sixteen levels
        const float u = ((float)(x & 0xFFFF) + (float)(x >> 16)) * (1.0f / 65536.0f) - 1.0f;
        p[i] = __float2half(u * amp);
    }
}
__global__ void fill_floats_kernel(float *p, size_t n, float v) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// Device buffers of one tuning run; everything is released when it goes out of scope.
struct Arena {
    std::vector<void *> ptrs;
    bool ok = true;
    template <typename T>
    T *get(size_t count) {
        void *p = nullptr;
        if (!ok || hipMalloc(&p, up(count * sizeof(T))) != hipSuccess) { ok = false; return nullptr; }
        ptrs.push_back(p);
        return static_cast<T *>(p);
    }
    ~Arena() { for (void *p : ptrs) (void)hipFree(p); }
};

unsigned fill_grid(size_t n) { const size_t b = (n + 255) / 256; return (unsigned)(b > 4096 ? 4096 : (b ? b : 1)); }

// A synthetic part: random codes in both precisions (any bits are a number in the FP6 layout, too), scales of the size trained
// layers have.
bool make_part(Arena &ar, int N, int K, int layout, int act, uint32_t seed, hipStream_t st, w4a4_part *out) {
    w4a4_part p = {};
    const size_t bytes4 = layout == W4A4_LAYOUT_FP6 ? (((size_t)N + 127) & ~(size_t)127) * (K / 4 * 3) : (size_t)N * (K / 2);
    uint8_t *q4 = ar.get<uint8_t>(bytes4);
    float *s4 = ar.get<float>(N);
    int32_t *es = ar.get<int32_t>(N);
    int8_t *q8 = ar.get<int8_t>((size_t)N * K);
    float *s8 = ar.get<float>(N);
    __half *bias = ar.get<__half>(N);
    if (!ar.ok) return false;
    hipLaunchKernelGGL(fill_bytes_kernel, dim3(fill_grid(bytes4 / 4)), dim3(256), 0, st, reinterpret_cast<uint32_t *>(q4), bytes4 / 4, seed);
    hipLaunchKernelGGL(fill_bytes_kernel, dim3(fill_grid((size_t)N * K / 4)), dim3(256), 0, st,
                       reinterpret_cast<uint32_t *>(q8), (size_t)N * K / 4, seed + 1);
    hipLaunchKernelGGL(fill_floats_kernel, dim3(fill_grid(N)), dim3(256), 0, st, s4, (size_t)N, 0.02f);
    hipLaunchKernelGGL(fill_floats_kernel, dim3(fill_grid(N)), dim3(256), 0, st, s8, (size_t)N, 0.001f);
    hipLaunchKernelGGL(fill_floats_kernel, dim3(fill_grid(N)), dim3(256), 0, st, reinterpret_cast<float *>(es), (size_t)N, 0.0f);
    hipLaunchKernelGGL(fill_halves_kernel, dim3(fill_grid(N)), dim3(256), 0, st, bias, (size_t)N, seed + 2, 0.1f);
    p.w4.q = q4; p.w4.scale = s4; p.w4.N = N; p.w4.K = K; p.w4.group = 0; p.w4.mode = W4A4_SYM;
    p.w4.layout = layout; p.w4.esum = layout == W4A4_LAYOUT_MFMA ? es : nullptr;
    p.w8q = q8; p.w8s = s8; p.bias_f16 = bias; p.act = act;
    *out = p;
    return true;
}

struct ShapeKey {
    int dev, M, h, ffn;
    bool operator<(const ShapeKey &o) const { return std::tie(dev, M, h, ffn) < std::tie(o.dev, o.M, o.h, o.ffn); }
};
std::mutex g_mu;
std::map<ShapeKey, int> g_tuned;

bool shape_ok(int M, int h, int ffn) {
    return M > 0 && h > 0 && ffn > 0 && h % 64 == 0 && ffn % 64 == 0 && h >= 128 && ffn >= 128 && h <= 4096 && ffn <= 16384;
}

}  // namespace
}  // namespace w4a4

using namespace w4a4;

extern "C" size_t w4a4_part_workspace_bytes(int M, const w4a4_part *P) {
    if (M <= 0 || !part_ok(P)) return 0;
    return part_bytes(M, *P);
}

extern "C" int w4a4_part_linear(const void *X_f16, int M, int ldx, const w4a4_part *P, int int4, void *out_f16,
                                void *workspace, size_t workspace_bytes, void *stream) {
    if (M < 0 || !part_ok(P) || ldx < P->w4.K) return W4A4_ERR_INVALID_ARG;
    if (M == 0) return W4A4_OK;
    if (!X_f16 || !out_f16) return W4A4_ERR_INVALID_ARG;
    if (!workspace || workspace_bytes < part_bytes(M, *P) || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return W4A4_ERR_WORKSPACE;
    return run_part(X_f16, M, ldx, *P, int4 != 0, out_f16, workspace, stream);
}

extern "C" size_t w4a4_ffn_workspace_bytes(int M, const w4a4_part *ffn1, const w4a4_part *ffn2) {
    if (M <= 0 || !part_ok(ffn1) || !part_ok(ffn2) || ffn1->w4.N != ffn2->w4.K) return 0;
    const size_t a = unfused_bytes(M, *ffn1, *ffn2);
    const size_t b = ffn2->w4.mode == W4A4_SYM ? plan_fused(nullptr, M, *ffn1, *ffn2).total : 0;
    return a > b ? a : b;
}

extern "C" int w4a4_ffn(const void *X_f16, int M, int ldx, const w4a4_part *ffn1, const w4a4_part *ffn2, int strategy,
                        void *out_f16, void *workspace, size_t workspace_bytes, void *stream) {
    if (M < 0 || !part_ok(ffn1) || !part_ok(ffn2) || ffn1->w4.N != ffn2->w4.K || ldx < ffn1->w4.K)
        return W4A4_ERR_INVALID_ARG;
    if (strategy < 0 || strategy > W4A4_STRATEGY_ALL_INT4) return W4A4_ERR_INVALID_ARG;
    const bool i1 = (strategy >> W4A4_PART_FFN1) & 1, i2 = (strategy >> W4A4_PART_FFN2) & 1;
    const bool fused = (strategy & W4A4_STRATEGY_FUSED_FFN) != 0;
    if (fused && !(i1 && i2)) return W4A4_ERR_INVALID_ARG;
    if (fused && ffn2->w4.mode != W4A4_SYM) return W4A4_ERR_UNSUPPORTED_SHAPE;
    // the FP6 kernel alone writes FP6 codes: a fused pair is in that layout on both sides or on neither
    if (fused && (ffn1->w4.layout == W4A4_LAYOUT_FP6) != (ffn2->w4.layout == W4A4_LAYOUT_FP6)) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if (M == 0) return W4A4_OK;
    if (!X_f16 || !out_f16) return W4A4_ERR_INVALID_ARG;
    if (!workspace || workspace_bytes < w4a4_ffn_workspace_bytes(M, ffn1, ffn2) ||
        (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1)))
        return W4A4_ERR_WORKSPACE;
    if (!fused) {
        uint8_t *H = static_cast<uint8_t *>(workspace);
        uint8_t *rest = H + up((size_t)M * ffn1->w4.N * 2);
        int rc = run_part(X_f16, M, ldx, *ffn1, i1, H, rest, stream);
        if (rc) return rc;
        return run_part(H, M, ffn1->w4.N, *ffn2, i2, out_f16, rest, stream);
    }
    const FusedPlan p = plan_fused(workspace, M, *ffn1, *ffn2);
    const w4a4_weight &w1 = ffn1->w4, &w2 = ffn2->w4;
    const w4a4_act a1 = view_act4(p.a1, M, w1.K, w1);
    int rc = w4a4_quantize_act(X_f16, M, w1.K, ldx, w1.mode, w1.group, p.a1.q, p.a1.scale, a1.zero ? p.a1.zero : nullptr,
                               a1.gsum ? p.a1.gsum : nullptr, w1.layout, p.a1.osum, stream);
    if (rc) return rc;
    const w4a4_epilogue ep1 = fused_epilogue(*ffn1, *ffn2);
    rc = w4a4_linear(&a1, &w1, &ep1, p.h.q, p.h.scale, nullptr, w2.layout == W4A4_LAYOUT_MFMA ? p.h.osum : nullptr,
                     p.lin_ws, p.lin_bytes, stream);
    if (rc) return rc;
    const w4a4_act h = view_act4(p.h, M, w2.K, w2);
    w4a4_epilogue ep2 = {};
    ep2.bias_f16 = ffn2->bias_f16;
    ep2.act = ffn2->act;
    return w4a4_linear(&h, &w2, &ep2, out_f16, nullptr, nullptr, nullptr, nullptr, 0, stream);
}

extern "C" int w4a4_strategy_pick(const w4a4_strategy_costs *c) {
    if (!c) return W4A4_ERR_INVALID_ARG;
    for (int p = 0; p < W4A4_PARTS; ++p)
        for (int k = 0; k < 2; ++k)
            if (!(c->part_us[p][k] >= 0.0f) || isinf(c->part_us[p][k])) return W4A4_ERR_INVALID_ARG;
    if (!(c->ffn_fused_us >= 0.0f) || isinf(c->ffn_fused_us)) return W4A4_ERR_INVALID_ARG;
    int best = -1, best_parts = -1, best_fused = -1;
    double best_cost = 0.0;
    for (int s = 0; s <= W4A4_STRATEGY_ALL_INT4; ++s) {
        const int b[4] = {s & 1, (s >> 1) & 1, (s >> 2) & 1, (s >> 3) & 1};
        const int fused = (s & W4A4_STRATEGY_FUSED_FFN) != 0;
        if (fused && !(b[2] && b[3])) continue;
        double cost = (double)c->part_us[0][b[0]] + (double)c->part_us[1][b[1]];
        cost += fused ? (double)c->ffn_fused_us : (double)c->part_us[2][b[2]] + (double)c->part_us[3][b[3]];
        const int parts = b[0] + b[1] + b[2] + b[3];
        const bool better = best < 0 || cost < best_cost ||
                            (cost == best_cost && (parts > best_parts || (parts == best_parts && fused > best_fused)));
        if (better) { best = s; best_cost = cost; best_parts = parts; best_fused = fused; }
    }
    return best;
}

extern "C" int w4a4_strategy_lookup(int M, int hidden, int ffn) {
    if (!shape_ok(M, hidden, ffn)) return W4A4_ERR_INVALID_ARG;
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess) {
        std::lock_guard<std::mutex> lock(g_mu);
        auto it = g_tuned.find(ShapeKey{dev, M, hidden, ffn});
        if (it != g_tuned.end()) return it->second;
    } else {
        (void)hipGetLastError();
    }
    // measured on MI355X for BERT-base and BERT-large shapes: INT4 wins every part at every token
    // count (by 2x and more below a few hundred tokens, where the INT4 part is one kernel); handing
    // the codes over in FFN1's epilogue beats a separate quantize of the fp16 intermediate only
    // for many tokens: from about 6144 at hidden size 1024, from about 16384 at 768.  Layer with weights in the layout it
    // takes, separate | fused, us: hidden 1024: 8192 tokens 166.2 | 164.4, 12288 239.6 | 227.9, 16384 291.0 | 284.8;
    // hidden 768: 12288 178.3 | 181.8, 14336 199.8 | 196.6, 16384 217.3 | 214.9, 20480 252.6 | 253.3, 24576 305.6 | 301.8
    const bool fused = hidden >= 1024 ? M >= 6144 : M >= 16384;
    return fused ? W4A4_STRATEGY_ALL_INT4 : 15;
}

extern "C" int w4a4_strategy_tune(int M, int hidden, int ffn, int iters, w4a4_strategy_costs *costs, void *stream) {
    if (!shape_ok(M, hidden, ffn) || iters <= 0 || iters > 1000) return W4A4_ERR_INVALID_ARG;
    hipStream_t st = as_stream(stream);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return W4A4_ERR_HIP;
    Arena ar;
    const int dims[4][2] = {{3 * hidden, hidden}, {hidden, hidden}, {ffn, hidden}, {hidden, ffn}};   // {N, K}
    w4a4_part parts[4];
    const bool fp6 = w4a4_encoder_layer_prefers_fp6(M, hidden, ffn) != 0;   // the INT4 kernels that a layer of this size runs on
    for (int p = 0; p < 4; ++p) {
        const int N = dims[p][0], K = dims[p][1], layout = fp6 ? W4A4_LAYOUT_FP6 : w4a4_preferred_layout(M, N, K, W4A4_SYM, 0);
        if (!make_part(ar, N, K, layout, p == W4A4_PART_FFN1 ? W4A4_ACT_GELU : W4A4_ACT_NONE, 1000u * (p + 1), st, &parts[p]))
            return W4A4_ERR_HIP;
    }
    const int widest = ffn > 3 * hidden ? ffn : 3 * hidden;
    __half *X = ar.get<__half>((size_t)M * widest);
    __half *Y = ar.get<__half>((size_t)M * widest);
    size_t ws_bytes = w4a4_ffn_workspace_bytes(M, &parts[2], &parts[3]);
    for (int p = 0; p < 4; ++p) {
        const size_t b = part_bytes(M, parts[p]);
        if (b > ws_bytes) ws_bytes = b;
    }
    uint8_t *ws = ar.get<uint8_t>(ws_bytes);
    if (!ar.ok) { (void)hipGetLastError(); return W4A4_ERR_HIP; }
    hipLaunchKernelGGL(fill_halves_kernel, dim3(fill_grid((size_t)M * widest)), dim3(256), 0, st, X, (size_t)M * widest, 7u, 3.0f);
    struct Events {
        hipEvent_t e[2] = {nullptr, nullptr};
        bool create() { return hipEventCreate(&e[0]) == hipSuccess && hipEventCreate(&e[1]) == hipSuccess; }
        ~Events() { for (hipEvent_t x : e) if (x) (void)hipEventDestroy(x); }
    } ev;
    if (!ev.create()) { (void)hipStreamSynchronize(st); return W4A4_ERR_HIP; }   // (the fills must finish before the arena goes)
    const hipEvent_t e0 = ev.e[0], e1 = ev.e[1];
    int status = W4A4_OK;
    auto time_us = [&](auto &&run, float *us) {
        if (status) return;
        for (int i = 0; i < 2 && !status; ++i) status = run();
        if (status) return;
        (void)hipEventRecord(e0, st);
        for (int i = 0; i < iters && !status; ++i) status = run();
        (void)hipEventRecord(e1, st);
        if (hipEventSynchronize(e1) != hipSuccess) { status = W4A4_ERR_HIP; return; }
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) { status = W4A4_ERR_HIP; return; }
        *us = ms * 1000.0f / (float)iters;
    };
    w4a4_strategy_costs c = {};
    for (int p = 0; p < 4; ++p)
        for (int k = 0; k < 2; ++k)
            time_us([&] { return run_part(X, M, dims[p][1], parts[p], k == 1, Y, ws, stream); }, &c.part_us[p][k]);
    time_us([&] { return w4a4_ffn(X, M, hidden, &parts[2], &parts[3], W4A4_STRATEGY_ALL_INT4, Y, ws, ws_bytes, stream); },
            &c.ffn_fused_us);
    (void)hipStreamSynchronize(st);
    if (status) return status;
    if (hipGetLastError() != hipSuccess) return W4A4_ERR_HIP;
    // Differences below 3 % are timing noise: price such options equally, so that the tie rules of the pick
    // (more INT4 parts, then the fused pair) decide and not the noise.  The caller gets the raw timings.
    w4a4_strategy_costs snapped = c;
    auto tie = [](float &a, float &b) {
        const float lo = a < b ? a : b, hi = a < b ? b : a;
        if (hi - lo <= 0.03f * lo) a = b = lo;
    };
    for (int p = 0; p < 4; ++p) tie(snapped.part_us[p][0], snapped.part_us[p][1]);
    {
        const float unfused = snapped.part_us[W4A4_PART_FFN1][1] + snapped.part_us[W4A4_PART_FFN2][1];
        if (snapped.ffn_fused_us > unfused && snapped.ffn_fused_us - unfused <= 0.03f * unfused) snapped.ffn_fused_us = unfused;
    }
    const int pick = w4a4_strategy_pick(&snapped);
    if (pick < 0) return pick;
    if (costs) *costs = c;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        g_tuned[ShapeKey{dev, M, hidden, ffn}] = pick;
    }
    return pick;
}

// Many tokens: the whole layer with its weights in the FP6 operand layout, if every part can take it (both FFN weights, so that
// the fused pair stays possible).  The FP6 kernels run the four GEMMs in less time once they fill the chip; below, their
// epilogue of separately rounded operations and the wider codes cost what the shorter main loop gives.  Layer in the layouts
// that w4a4_preferred_layout names | in FP6, sequences of 128, built-in strategy, us: hidden 1024: 6144 tokens 137 | 141,
// 8192 171 | 166, 12288 242 | 227, 16384 310 | 283; hidden 768: 8192 130 | 134, 12288 181 | 178, 16384 230 | 216, 24576 315 | 300.
// Not at 512 features, where short K leaves the wider codes nothing to win (12288 tokens 113 | 125, 24576 191 | 194), nor past 3072, where
// the int8 kernel's 256 x 256 tiles make up for it (4096, ffn 8192: 8192 tokens 956 | 1037, 16384 1833 | 1877, 24576 2730 | 2746).  Between:
// 1280 12288 tokens 342 | 307, 2048 636 | 616, 2560 696 | 658, 3072 (ffn 6144) 8192 642 | 650, 12288 950 | 893, 16384 1182 | 1169, 24576 1797 | 1719.
extern "C" int w4a4_encoder_layer_prefers_fp6(int M, int hidden, int ffn) {
    if (!shape_ok(M, hidden, ffn) || hidden < 768 || hidden > 3072 || M < (hidden >= 1024 ? 8192 : 12288)) return 0;
    int lpr = 0, opl = 0;
    for (int k : {hidden, ffn})
        if (k % 128 || k < 512 || !fp6_plan(k, &lpr, &opl)) return 0;
    const int widest = ffn > 3 * hidden ? ffn : 3 * hidden;
    // sizes the FP6 kernel addresses with 32 bits, and FFN1's requantized output: whole column tiles that fit side by side
    if (((long)M + 512) * widest * 4 >= 0x80000000L || ((long)widest + 128) * (widest / 4 * 3) >= 0x7fffffffL || ffn % 256) return 0;
    return ffn / 256 <= fp6_requant_max_tiles_n() ? 1 : 0;
}

extern "C" size_t w4a4_encoder_layer_workspace_bytes(int batch, int seq, const w4a4_encoder_layer_weights *L) {
    if (batch <= 0 || seq <= 0 || (long)batch * seq > 0x7fffffffL / 4 || !layer_ok(L)) return 0;
    return plan_layer(nullptr, batch * seq, *L).total;
}

extern "C" int w4a4_encoder_layer(const void *X_f16, int batch, int seq, const w4a4_encoder_layer_weights *L, int strategy,
                                  void *out_f16, void *workspace, size_t workspace_bytes, void *stream) {
    if (batch < 0 || seq < 0 || (long)batch * seq > 0x7fffffffL / 4 || !layer_ok(L)) return W4A4_ERR_INVALID_ARG;
    if (strategy < 0 || strategy > (W4A4_STRATEGY_ALL_INT4 | W4A4_STRATEGY_FUSED_LN)) return W4A4_ERR_INVALID_ARG;
    const bool i0 = strategy & 1, i1 = (strategy >> 1) & 1, i2 = (strategy >> 2) & 1, i3 = (strategy >> 3) & 1;
    const bool fused_ffn = (strategy & W4A4_STRATEGY_FUSED_FFN) != 0, fused_ln = (strategy & W4A4_STRATEGY_FUSED_LN) != 0;
    if ((fused_ffn && !(i2 && i3)) || (fused_ln && !i2)) return W4A4_ERR_INVALID_ARG;
    const int M = batch * seq;
    if (M == 0) return W4A4_OK;
    if (!X_f16 || !out_f16) return W4A4_ERR_INVALID_ARG;
    if (seq > 512) return W4A4_ERR_UNSUPPORTED_SHAPE;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kAlign - 1))) return W4A4_ERR_WORKSPACE;
    const LayerPlan p = plan_layer(workspace, M, *L);
    if (workspace_bytes < p.total) return W4A4_ERR_WORKSPACE;
    const int h = L->hidden;
    const w4a4_weight &w1 = L->ffn1.w4, &w2 = L->ffn2.w4;

    int rc = run_part(X_f16, M, h, L->qkv, i0, p.qkv, p.rest, stream);
    if (rc) return rc;
    rc = w4a4_attention_f16(p.qkv, batch, seq, L->heads, p.ctx, stream);
    if (rc) return rc;
    rc = run_part(p.ctx, M, h, L->attn_out, i1, p.ao, p.rest, stream);
    if (rc) return rc;
    // x1 = LN1(attn_out + x).  Where FFN1 reads INT4 codes from memory, the same kernel writes them: of LayerNorm's fp32
    // result (fused_ln), or of x1 itself, what w4a4_quantize_act would make of it.  It also clears what FFN1's
    // requantizing epilogue counts in.  (16384 tokens of 768, layer: 247 us with the separate quantize and fill launches
    // and LayerNorm 2 writing codes that nothing reads, 233 us so; 465 tokens: 49.6 and 44.3 us.)
    const bool from_codes = fused_ln || (i2 && (fused_ffn || !one_kernel_ffn1(M, w1)));
    const w4a4_act a1 = view_act4(p.ln, M, h, w1);
    Carver c(p.rest);
    ActBuffers hb = {};
    w4a4_epilogue ep1 = {};
    size_t lin_bytes = 0;
    void *lin_ws = nullptr;
    int32_t *h_osum = nullptr;
    ClearRanges clear = {};
    if (from_codes && fused_ffn) {
        if (w2.mode != W4A4_SYM || (w1.layout == W4A4_LAYOUT_FP6) != (w2.layout == W4A4_LAYOUT_FP6)) return W4A4_ERR_UNSUPPORTED_SHAPE;
        hb = carve_act4(c, M, w2.K, w2);
        h_osum = w2.layout == W4A4_LAYOUT_MFMA ? hb.osum : nullptr;
        ep1 = fused_epilogue(L->ffn1, L->ffn2);
        lin_bytes = w4a4_linear_workspace_bytes(&a1, &w1, &ep1, h_osum != nullptr);
        lin_ws = c.take<uint8_t>(lin_bytes);
        clear = linear_clear_ranges(&a1, &w1, &ep1, h_osum, lin_ws);
    }
    // Few tokens: FFN1's kernel quantizes its tokens' whole rows itself, so it forms LayerNorm 1 of them first, one launch less
    // (layer of 768 at 1 x 32 tokens 29.0 -> 26.7 us, 1 x 128 33.3 -> 31.8; of 1024 at 1 x 128 35.8 -> 34.7).
    const LnArgs ln1 = layernorm_args(p.ao, X_f16, M, h, L->ln1_gamma_f16, L->ln1_beta_f16, L->ln_eps, p.x1);
    __half *H = nullptr;
    if (!fused_ffn) {
        H = c.take<__half>((size_t)M * w1.N);
        ep1.bias_f16 = L->ffn1.bias_f16;
        ep1.act = L->ffn1.act;
    }
    const bool ln_in_ffn1 = i2 && !from_codes && linear_layernorm_f16act_ok(ln1, w1, ep1, H);
    if (!ln_in_ffn1) {
        rc = run_layernorm(p.ao, X_f16, M, h, L->ln1_gamma_f16, L->ln1_beta_f16, L->ln_eps, p.x1, p.ln, w1.layout,
                           !from_codes ? LN_CODES_NONE : fused_ln ? LN_CODES_F32 : LN_CODES_F16, clear, stream);
        if (rc) return rc;
    }
    if (ln_in_ffn1) {
        rc = linear_layernorm_f16act(ln1, w1, ep1, H, as_stream(stream));
        if (rc) return rc;
        rc = run_part(H, M, w1.N, L->ffn2, i3, p.h2, p.rest + c.used, stream);
        if (rc) return rc;
    } else if (!from_codes) {
        rc = w4a4_ffn(p.x1, M, h, &L->ffn1, &L->ffn2, strategy & W4A4_STRATEGY_ALL_INT4, p.h2, p.rest, p.rest_bytes, stream);
        if (rc) return rc;
    } else if (fused_ffn) {
        rc = linear_cleared(&a1, &w1, &ep1, hb.q, hb.scale, h_osum, lin_ws, lin_bytes, stream);
        if (rc) return rc;
        const w4a4_act hv = view_act4(hb, M, w2.K, w2);
        w4a4_epilogue ep2 = {};
        ep2.bias_f16 = L->ffn2.bias_f16;
        ep2.act = L->ffn2.act;
        rc = w4a4_linear(&hv, &w2, &ep2, p.h2, nullptr, nullptr, nullptr, nullptr, 0, stream);
        if (rc) return rc;
    } else {
        rc = w4a4_linear(&a1, &w1, &ep1, H, nullptr, nullptr, nullptr, nullptr, 0, stream);
        if (rc) return rc;
        rc = run_part(H, M, w1.N, L->ffn2, i3, p.h2, p.rest + c.used, stream);
        if (rc) return rc;
    }
    // out = LN2(ffn2 + x1)
    return run_layernorm(p.h2, p.x1, M, h, L->ln2_gamma_f16, L->ln2_beta_f16, L->ln_eps, out_f16, ActBuffers{},
                         W4A4_LAYOUT_CANONICAL, LN_CODES_NONE, ClearRanges{}, stream);
}
