// What the host code that composes an encoder layer uses of the LayerNorm kernel and of w4a4_linear beside the C ABI.
#pragma once
#include "common.hpp"

namespace w4a4 {

struct LnArgs {
    const __half *X, *R; long ldx;       // [M, ldx] each; R may be NULL
    const __half *gamma, *beta;          // [K]
    float eps;
    __half *Y;                           // [M, K] or NULL
    uint8_t *q; float *s, *z;            // [M, K/2], [M], [M]
    int32_t *gsum; int ng, cpg;          // [M, ng] code sums of runs of cpg chunks (NULL = not wanted)
    int32_t *psum;                       // [M] odd-position code sums (MFMA operand layout)
    int M, K;
    uint32_t *zero0, *zero1; int n0, n1; // words the kernel clears besides: counters of a later kernel on the stream
};

// What the token-wise quantize works on: nothing (no codes, q and s unused), the fp32 result of the LayerNorm, or its
// fp16 copy, i.e. what w4a4_quantize_act would make of Y.
enum LnCodes { LN_CODES_NONE, LN_CODES_F32, LN_CODES_F16 };

// Launches the kernel for symmetric codes in `layout`; the caller has checked the arguments as w4a4_layernorm_quantize does.
int layernorm_rows(const LnArgs &a, int layout, int codes, hipStream_t st);

// w4a4_linear_f16act on the fp16 result of a LayerNorm with residual, which is formed in the same launch and goes to ln.Y (ln.q and the
// code sums are not used).  Symmetric per-channel weights in the canonical layout; _ok: the sizes and pointers it takes.
bool linear_layernorm_f16act_ok(const LnArgs &ln, const w4a4_weight &W, const w4a4_epilogue &ep, const void *out);
int linear_layernorm_f16act(const LnArgs &ln, const w4a4_weight &W, const w4a4_epilogue &ep, void *out, hipStream_t st);

// Whether the kernel of w4a4_linear_f16act has K as a constant (some 30 % less time than with K at run time).
bool small_constant_k(int K);

// Words that a requantizing w4a4_linear needs cleared (none if its requantize is not fused), and that call for a caller
// whose previous kernel on the stream has cleared them.
struct ClearRanges { uint32_t *p0, *p1; int n0, n1; };
ClearRanges linear_clear_ranges(const w4a4_act *A, const w4a4_weight *W, const w4a4_epilogue *ep, int32_t *out_gsum, void *workspace);
int linear_cleared(const w4a4_act *A, const w4a4_weight *W, const w4a4_epilogue *ep, void *out, float *out_scale,
                   int32_t *out_gsum, void *workspace, size_t workspace_bytes, void *stream);

// Column tiles of a row panel that the FP6 kernel's requantizing epilogue can keep co-resident (-1: HIP error).
int fp6_requant_max_tiles_n();

}  // namespace w4a4
