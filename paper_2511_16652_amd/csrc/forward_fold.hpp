// Pieces of the forward layer shared by its translation units: the bf16-grade GELU, the flags of the store-only epilogues and
// the launch interface of the folded layer (k_forward_fold.hip).
#pragma once
#include "common.hpp"

namespace egg {

// What a store-only epilogue does behind the accumulators, fixed at compile time (LEAN_PROJ: k_forward.hip)
enum { LEAN_ON = 1, LEAN_GELU = 2, LEAN_RESID = 4, LEAN_PROJ = 8 };

// gelu(x) = x Phi(x) for outputs that are rounded to bf16.  Every vector-ALU slot of the epilogue is exposed time
// (one slot per element costs about 1 % of a K = 2048 tile), and the library erff costs about 27 of them.  Here
// Phi(x) - 1/2 is an odd degree-17 polynomial on [-4, 4] (least squares on Chebyshev nodes, pinned to 1/2 at the
// ends so that the clamp continues it with Phi = 0 and Phi = 1): 12 slots.  |error of gelu| <= 2e-5 inside
// (-3.8, 3.8) and <= 1.3e-4 at |x| = 4 (the neglected tail 4 Phi(-4)); a bf16 ulp of gelu is larger than that
// wherever |gelu(x)| > 0.03.  fp32 outputs keep erff.
// Four values at a time, step by step, so that the four Horner chains are independent neighbours in the
// instruction stream (a dependent fma cannot issue back to back).
__device__ __forceinline__ void gelu_bf16_grade4(float (&y)[4])
{
    float xc[4], x2[4], p[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) xc[e] = __builtin_amdgcn_fmed3f(y[e], -4.0f, 4.0f);
#pragma unroll
    for (int e = 0; e < 4; ++e) x2[e] = xc[e] * xc[e];
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = fmaf(8.809068429e-11f, x2[e], -7.454938351e-09f);
#define EGG_GELU_STEP(C) _Pragma("unroll") for (int e = 0; e < 4; ++e) p[e] = fmaf(p[e], x2[e], C);
    EGG_GELU_STEP(2.826503707e-07f)
    EGG_GELU_STEP(-6.433988670e-06f)
    EGG_GELU_STEP(9.985887631e-05f)
    EGG_GELU_STEP(-1.137293224e-03f)
    EGG_GELU_STEP(9.882503528e-03f)
    EGG_GELU_STEP(-6.641100396e-02f)
    EGG_GELU_STEP(3.989198364e-01f)
#undef EGG_GELU_STEP
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] *= fmaf(xc[e], p[e], 0.5f);
}

// The parts of the N products c t that a fold's K-slots hold: the nearest bf16 values or what they leave, which together are c t to about
// 2^-17; the layer's output is rounded to bf16, 2^-9, behind it.  Measured against 64 bits over ranks 1 to 16, 16 to 200 rows per member,
// 512 x 512 and 1024 -> 2048 (relative 2-norm, 1.66e-3 throughout), the correction folded / in fp32: at sigma = 0.001 the same in
// seven digits, at sigma = 0.5, where the correction is of the output's size, larger by 1.2e-6 of itself (2.4e-6 at most).
// A finite c t that would round to infinity takes the largest bf16 value, and an infinite one leaves nothing (inf - inf is NaN): the
// products with the factors are then those of c t itself.  The operations are written out, none is left to contraction: a member's
// bits are the same in every kernel that folds.
template <int N>
__device__ __forceinline__ void bf16_parts(float c, const float (&t)[N], bool rest, float (&out)[N])
{
#pragma clang fp contract(off)
    float top = 0.f;
#pragma unroll
    for (int l = 0; l < N; ++l) {
        const float x = c * t[l], hi = round_bf16(x);
        out[l] = rest ? fmaf(c, t[l], -hi) : hi;
        top = fmaxf(top, fabsf(x));
    }
    const float most = __uint_as_float(0x7F7F0000u);
    if (__any(top > most)) {
#pragma unroll
        for (int l = 0; l < N; ++l) {
            const float x = c * t[l];
            if (fabsf(x) > most) {
                const float hi = __builtin_isinf(x) ? x : __builtin_copysignf(most, x);
                out[l] = !rest ? hi : (__builtin_isinf(x) ? 0.f : x - hi);
            }
        }
    }
}

// One bf16 layer whose correction is folded into the accumulators as a few more MFMAs (or is off: c = 0), for every shape
// that the parked form of k_forward.hip does not take: S not a multiple of 64, rank 16, ragged K, few tiles.
struct FoldLayer {
    int S;            // rows per noise id (a pair's 2S rows count as one member's); at least FOLD_MIN_ROWS when c != 0
    int d_out, d_in, rank;
    int64_t R;
    float c;          // sigma / sqrt(rank)
    bool gelu;
    const void *W, *X, *A, *resid;  // A: materialised factors [id][d_out][rank] bf16; resid may be NULL
    void* Y;
    const float* t;
};
constexpr int FOLD_MIN_ROWS = 15;  // 16 neighbouring rows then belong to at most two members
egg_status launch_forward_fold(eggroll_ctx* c, const FoldLayer& l);

}  // namespace egg
