// Version and status strings of libw4a4, the timing hook, calls laid out once.
#include "common.hpp"

extern "C" const char *w4a4_version(void) { return "w4a4 0.1 (gfx950)"; }

extern "C" const char *w4a4_status_string(int status) {
    switch (status) {
        case W4A4_OK: return "ok";
        case W4A4_ERR_INVALID_ARG: return "invalid argument";
        case W4A4_ERR_UNSUPPORTED_SHAPE: return "unsupported shape or alignment";
        case W4A4_ERR_WORKSPACE: return "workspace missing or too small";
        case W4A4_ERR_HIP: return "HIP launch failed";
        default: return "unknown status";
    }
}

namespace w4a4 {
KernelTimer &kernel_timer() {
    static thread_local KernelTimer t;
    return t;
}
}  // namespace w4a4

extern "C" int w4a4_time_next_gemm(void *start_event, void *stop_event) {
    w4a4::KernelTimer &t = w4a4::kernel_timer();
    t.start = reinterpret_cast<hipEvent_t>(start_event);
    t.stop = reinterpret_cast<hipEvent_t>(stop_event);
    return W4A4_OK;
}

extern "C" int w4a4_run_call(const w4a4_call *c, void *st) {
    if (!c) return W4A4_ERR_INVALID_ARG;
    void *const *p = c->p;
    const int *i = c->i;
    auto u8 = [&](int k) { return static_cast<uint8_t *>(p[k]); };
    auto i8 = [&](int k) { return static_cast<int8_t *>(p[k]); };
    auto i32 = [&](int k) { return static_cast<int32_t *>(p[k]); };
    auto f32 = [&](int k) { return static_cast<float *>(p[k]); };
    auto ep = [&](int k) { return static_cast<const w4a4_epilogue *>(p[k]); };
    auto weight = [&](int k) { return static_cast<const w4a4_weight *>(p[k]); };
    switch (c->entry) {
        case W4A4_CALL_QUANTIZE_ACT:
            return w4a4_quantize_act(p[0], i[0], i[1], i[2], i[3], i[4], u8(1), f32(2), f32(3), i32(4), i[5], i32(5), st);
        case W4A4_CALL_LINEAR:
            return w4a4_linear(static_cast<const w4a4_act *>(p[0]), weight(1), ep(2), p[3], f32(4), f32(5), i32(6), p[7], c->n, st);
        case W4A4_CALL_LINEAR_F16ACT:
            return w4a4_linear_f16act(p[0], i[0], i[1], i[2], weight(1), ep(2), p[3], st);
        case W4A4_CALL_LAYERNORM_QUANTIZE:
            return w4a4_layernorm_quantize(p[0], p[1], i[0], i[1], i[2], p[2], p[3], c->f, p[4], i[3], i[4], u8(5), f32(6), f32(7), i32(8), i[5], i32(9), st);
        case W4A4_CALL_QUANTIZE_ROWS8:
            return w8a8_quantize_rows(p[0], i[0], i[1], i[2], i8(1), f32(2), st);
        case W4A4_CALL_LINEAR8:
            return w8a8_linear(i8(0), i[0], f32(1), i[1], i8(2), f32(3), i[2], i[3], ep(4), p[5], st);
        default: return W4A4_ERR_INVALID_ARG;
    }
}
