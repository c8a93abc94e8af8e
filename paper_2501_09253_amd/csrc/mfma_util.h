// Types and small device helpers shared by the bf16 matrix-core kernels.
#pragma once

#include "kernels.h"

namespace pserve {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// GELU(v) = v/2 (1 + erf(v/sqrt 2)) with erf from the 5-term rational-exponential form (Abramowitz & Stegun
// 7.1.26, |error| < 1.5e-7): far below the bf16 resolution of the output and several times cheaper than erff.
// With u = |v|, t = 1/(1 + p u/sqrt 2) and y = (a1 t + .. + a5 t^5)/2 * exp(-u^2/2):  erf(u/sqrt 2) = 1 - 2y, so
// GELU(v) = v (1 - y) for v >= 0 and v y for v < 0.  Hardware reciprocal and exp2 (1 ulp each); 15 instructions.
__device__ __forceinline__ float gelu_erf(float v) {
    const float u = fabsf(v);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, u, 1.f));
    float p = fmaf(0.5f * 1.061405429f, t, 0.5f * -1.453152027f);
    p = fmaf(p, t, 0.5f * 1.421413741f);
    p = fmaf(p, t, 0.5f * -0.284496736f);
    p = fmaf(p, t, 0.5f * 0.254829592f);
    const float y = p * t * __builtin_amdgcn_exp2f(u * u * (-0.5f * 1.4426950408889634f));
    const float r = v * y;
    return v >= 0.f ? v - r : r;
}

// GELU, tanh form: v/2 (1 + tanh(u)) = v / (1 + exp(-2u)), u = sqrt(2/pi) (v + 0.044715 v^3); hardware exp2 and reciprocal
__device__ __forceinline__ float gelu_tanh(float v) {
    const float u2 = v * fmaf(0.044715f * v, v, 1.f) * (-2.f * 0.7978845608028654f * 1.4426950408889634f);   // -2u log2(e)
    return v * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(u2));
}

// value of lane l ^ 32 (v_permlane32_swap: upper half of the first operand <-> lower half of the second)
__device__ __forceinline__ float other_half_f(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float((threadIdx.x & 32) ? r[0] : r[1]);
}

typedef __attribute__((address_space(3))) void lds_void;

// Text rows stand L to a request and their outputs row_group_pad apart.  A transposed segment stores four tokens at once
// where they lie aligned; with L = 77 and 80 only every fourth request's do, and the others' leave two bytes at a time.  The
// tiles then walk the padded rows instead (those past L hold nothing): 39 -> 33 us for 22 x 77 x 2560, K = 2048; 16 requests
// 30.7 -> 26.1, 10 29.1 -> 24.5, 4 19.8 -> 19.2; 4 x 77 x 1280, K = 768 13.5 -> 12.1, but 2 11.7 -> 12.1.  Not where the padding
// would be more than an eighth of the rows, nor where L is a multiple of four or there are fewer than three requests.  A form of
// its own (EPF_PADS): as a run-time choice in all forms it cost the small layers 2 to 10 % (1,024 x 1,280, K = 1,280 and 128 x 64
// tiles 12.5 -> 13.0 .. 13.7 us).
__host__ __device__ inline bool gemm_pads_rows(const GemmArgs& a) {
    return !a.tokens_are_rows && a.epi == EPI_ROUTE && !a.rowbias && !a.rowscale && !a.act_gelu && a.row_group > 0 &&
           a.M > 2 * a.row_group && a.row_group % 4 != 0 && a.row_group_pad % 4 == 0 && a.M % a.row_group == 0 &&
           a.row_group_pad - a.row_group <= a.row_group / 8 && (a.seg[0].transposed || a.seg[1].transposed || a.seg[2].transposed);
}
// problems the bf16 MFMA kernels take at all
inline bool gemm_mfma_eligible(const GemmArgs& a) {
    return a.K % 64 == 0 && a.lda % 8 == 0 && !((uintptr_t)a.A & 15) && !((uintptr_t)a.B & 15) && gemm_fits32(a);
}
// second problems the kernels with one tile a block take
inline bool gemm_two_eligible(const GemmArgs& a) {
    return a.epi == EPI_ROUTE && !a.conv && a.tokens_are_rows && a.act.active && a.act2.active && !((uintptr_t)a.B2 & 15) &&
           !a.bias == !a.bias2 && !a.rowscale == !a.rowscale2 && !a.rowbias;
}
// Token of the unpadded batch that holds pixel (Y, X) of patch p's padded layout (GemmArgs::halo_src), -1: outside the image
__device__ __forceinline__ int halo_token(const GemmArgs& a, int p, int Y, int X) {
    const int ppw = a.geom.ppw, pw = ppw - 2, ph = a.geom.pS / ppw - 2;
    if (Y >= 1 && Y <= ph && X >= 1 && X <= pw) return p * (ph * pw) + (Y - 1) * pw + X - 1;
    return a.halo_src[p * (2 * ppw + 2 * ph) + (Y < 1 ? X : Y > ph ? ppw + X : 2 * ppw + (X < 1 ? 0 : ph) + Y - 1)];
}
// its byte offset; past the tensor's end, where buffer loads give zeros, for pixels outside the image
__device__ __forceinline__ int halo_offset(const GemmArgs& a, int tok) { return tok < 0 ? 0x7fffff00 : (int)((int64_t)tok * a.lda * 2); }
// bytes of the unpadded batch
__device__ __forceinline__ int halo_bytes(const GemmArgs& a) {
    const int ppw = a.geom.ppw;
    return (int)((int64_t)a.geom.P * (a.geom.pS / ppw - 2) * (ppw - 2) * a.lda * 2);
}
__host__ __device__ inline int32_t gemm_rows(const GemmArgs& a) { return gemm_pads_rows(a) ? a.M / a.row_group * a.row_group_pad : a.M; }

}  // namespace pserve
