// Device helpers shared by the kernels of the linear layer: vector types, the GELU forms, bf16
// conversion and the epilogue of output elements.
#pragma once

#include "tess_internal.h"

#include <type_traits>

namespace tess {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(T) __attribute__((address_space(3))) T*


// Compile-time loop: the body sees the index as an integral constant, so every
// accumulator index is static and the accumulators stay in registers.
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// ---------------------------------------------------------------------------
// epilogue helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ float gelu_erf_f(float x)
{
    return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f));
}
// GELU (erf form) for 2-byte outputs, branch-free and about half the instructions of
// the library erf: with z = |x|/sqrt(2) and t = 1/(1 + p z), the rational-exponential
// approximation of Abramowitz & Stegun 7.1.26 gives erfc(z) = poly(t) exp(-z^2) with
// absolute error below 1.5e-7.  1 + erf(x/sqrt(2)) is erfc(z) for x < 0 (no cancellation
// in the tail) and 2 - erfc(z) otherwise.
__device__ __forceinline__ float gelu_erf_fast(float x)
{
    const float z = __builtin_fabsf(x) * 0.70710678118654752440f;
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, z, 1.0f));
    float p = __builtin_fmaf(1.061405429f, t, -1.453152027f);
    p = __builtin_fmaf(p, t, 1.421413741f);
    p = __builtin_fmaf(p, t, -0.284496736f);
    p = __builtin_fmaf(p, t, 0.254829592f);
    const float e = __builtin_amdgcn_exp2f(x * x * -0.72134752044448170368f);   // exp(-x^2/2)
    const float erfc_z = p * t * e;
    const float one_plus_erf = x < 0.0f ? erfc_z : 2.0f - erfc_z;
    return 0.5f * x * one_plus_erf;
}
__device__ __forceinline__ float gelu_tanh_f(float x)
{
    const float c = 0.79788456080286535588f;
    return 0.5f * x * (1.0f + tanhf(c * (x + 0.044715f * x * x * x)));
}
// Derivatives: d/dx [x Phi(x)] = Phi(x) + x phi(x); for the tanh form the chain rule on
// u = c (x + 0.044715 x^3).
__device__ __forceinline__ float gelu_erf_grad_f(float x)
{
    const float Phi = 0.5f * (1.0f + erff(x * 0.70710678118654752440f));
    return Phi + x * 0.39894228040143267794f * __expf(-0.5f * x * x);
}
__device__ __forceinline__ float gelu_tanh_grad_f(float x)
{
    const float c = 0.79788456080286535588f;
    const float th = tanhf(c * (x + 0.044715f * x * x * x));
    return 0.5f * (1.0f + th) + 0.5f * x * (1.0f - th * th) * c * (1.0f + 0.134145f * x * x);
}
// The same erfc form as gelu_erf_fast; its exponential is the normal density up to a factor.
__device__ __forceinline__ float gelu_erf_grad_fast(float x)
{
    const float z = __builtin_fabsf(x) * 0.70710678118654752440f;
    const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3275911f, z, 1.0f));
    float p = __builtin_fmaf(1.061405429f, t, -1.453152027f);
    p = __builtin_fmaf(p, t, 1.421413741f);
    p = __builtin_fmaf(p, t, -0.284496736f);
    p = __builtin_fmaf(p, t, 0.254829592f);
    const float e = __builtin_amdgcn_exp2f(x * x * -0.72134752044448170368f);   // exp(-x^2/2)
    const float erfc_z = p * t * e;
    const float one_plus_erf = x < 0.0f ? erfc_z : 2.0f - erfc_z;
    return __builtin_fmaf(x * 0.39894228040143267794f, e, 0.5f * one_plus_erf);
}
__device__ __forceinline__ float apply_act_grad(float z, int act)
{
    if (act == TESS_ACT_GELU_ERF) return gelu_erf_grad_f(z);
    if (act == TESS_ACT_GELU_TANH) return gelu_tanh_grad_f(z);
    return 1.0f;
}
__device__ __forceinline__ float apply_act(float z, int act)
{
    if (act == TESS_ACT_GELU_ERF) return gelu_erf_f(z);
    if (act == TESS_ACT_GELU_TANH) return gelu_tanh_f(z);
    return z;
}
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b)
{
    return __uint_as_float(((uint32_t)b) << 16);
}
__device__ __forceinline__ float load_in(const void* p, int64_t idx, int in_f32)
{
    return in_f32 ? ((const float*)p)[idx] : bf16_bits_to_f32(((const uint16_t*)p)[idx]);
}

// four fp32 -> four bf16 (round to nearest even, the hardware conversion of gfx950)
__device__ __forceinline__ u32x2 pack_bf16x4(floatx4 v)
{
    const floatx2 lo = {v[0], v[1]}, hi = {v[2], v[3]};
    u32x2 w;
    w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
    w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
    return w;
}

enum : int { MODE_BF16 = 0, MODE_BF16_GELU = 1, MODE_F32 = 2, MODE_F32_ACC = 3, MODE_GENERIC = 4,
             MODE_BF16_DGELU = 5, MODE_BF16_GELU_PRE = 6 };


// Epilogue for four adjacent columns of one output row: bias, optional copy of the
// pre-activation, activation, then store or accumulate in the output dtype.  `vec`:
// rows are 16-byte aligned, so the four values go out as one store.  The mode flags
// are template parameters so that the drain loop of the common cases is a handful of
// instructions; MODE_GENERIC reads them from the arguments instead.
template <int MODE>
__device__ __forceinline__ void emit4(const GemmArgs& g, int row, int col, floatx4 v, floatx4 bias,
                                      bool vec, u32x2 zbits = u32x2{0u, 0u})
{
    const bool out_f32 = MODE == MODE_GENERIC ? (g.out_f32 != 0) : (MODE == MODE_F32 || MODE == MODE_F32_ACC);
    const bool accumulate = MODE == MODE_GENERIC ? (g.accumulate != 0) : (MODE == MODE_F32_ACC);
    // MODE_BF16_GELU_PRE: the MLP up-projection that keeps its pre-activation for the backward
    // pass; same GELU evaluation as MODE_BF16_GELU, so the layer's output does not depend on
    // whether the pre-activation is asked for
    const bool preact = MODE == MODE_GENERIC ? (g.preact != nullptr) : (MODE == MODE_BF16_GELU_PRE);
    const int act = MODE == MODE_GENERIC ? g.act
                    : ((MODE == MODE_BF16_GELU || MODE == MODE_BF16_GELU_PRE) ? TESS_ACT_GELU_ERF : TESS_ACT_NONE);
    const int nvalid = g.N - col < 4 ? g.N - col : 4;
    v += bias;
    const int64_t o = (int64_t)row * g.ldo + col;
    const bool full = vec && nvalid == 4;
    if (preact) {
        if (out_f32) {
            float* p = (float*)g.preact + o;
            if (full) *(floatx4*)p = v;
            else for (int e = 0; e < nvalid; ++e) p[e] = v[e];
        } else {
            uint16_t* p = (uint16_t*)g.preact + o;
            const u32x2 w = pack_bf16x4(v);
            if (full) *(u32x2*)p = w;
            else for (int e = 0; e < nvalid; ++e) p[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
        }
    }
    if (MODE == MODE_BF16_DGELU) {
        // zbits: the bf16 pre-activations of the same four columns, fetched by the caller
        // ahead of time (elements past the edge are zero and their products are not stored)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] *= gelu_erf_grad_fast(__uint_as_float((e & 1) ? (zbits[e >> 1] & 0xffff0000u) : (zbits[e >> 1] << 16)));
    } else if (MODE == MODE_GENERIC && g.zin) {
        for (int e = 0; e < nvalid; ++e)
            v[e] *= apply_act_grad(load_in(g.zin, (int64_t)row * g.ldz + col + e, g.in_f32), g.dact);
    }
    if (act != TESS_ACT_NONE) {
        // every 2-byte erf-GELU output takes the same evaluation, whichever kernel or drain
        // produces it; fp32 outputs take the library erf
        if (MODE == MODE_BF16_GELU || MODE == MODE_BF16_GELU_PRE ||
            (MODE == MODE_GENERIC && !out_f32 && act == TESS_ACT_GELU_ERF)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_erf_fast(v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = apply_act(v[e], act);
        }
    }
    if (out_f32) {
        float* p = (float*)g.out + o;
        if (full) {
            if (accumulate) v += *(const floatx4*)p;
            __builtin_nontemporal_store(v, (floatx4*)p);       // written once, not read again here
        } else {
            for (int e = 0; e < nvalid; ++e) p[e] = accumulate ? p[e] + v[e] : v[e];
        }
    } else {
        uint16_t* p = (uint16_t*)g.out + o;
        const u32x2 w = pack_bf16x4(v);
        if (full) __builtin_nontemporal_store(w, (u32x2*)p);   // streaming store: +1-2 % on the forward calls
        else for (int e = 0; e < nvalid; ++e) p[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
    }
}

// Eight adjacent columns of one output row in one of the 2-byte output modes: the same
// arithmetic as two emit4 calls, but the row leaves as one 16-byte store per lane (and the
// pre-activation as another) when all eight columns exist and the rows are 16-byte aligned.
template <int MODE>
__device__ __forceinline__ void emit8_bf16(const GemmArgs& g, int row, int col, floatx4 v0, floatx4 v1,
                                           floatx4 b0, floatx4 b1, bool vec)
{
    static_assert(MODE == MODE_BF16 || MODE == MODE_BF16_GELU || MODE == MODE_BF16_GELU_PRE, "2-byte outputs");
    if (!(vec && col + 8 <= g.N)) {
        emit4<MODE>(g, row, col, v0, b0, vec);
        if (col + 4 < g.N) emit4<MODE>(g, row, col + 4, v1, b1, vec);
        return;
    }
    v0 += b0;
    v1 += b1;
    const int64_t o = (int64_t)row * g.ldo + col;
    if (MODE == MODE_BF16_GELU_PRE) {
        const u32x2 p0 = pack_bf16x4(v0), p1 = pack_bf16x4(v1);
        __builtin_nontemporal_store(u32x4{p0[0], p0[1], p1[0], p1[1]}, (u32x4*)((uint16_t*)g.preact + o));
    }
    if (MODE != MODE_BF16) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v0[e] = gelu_erf_fast(v0[e]); v1[e] = gelu_erf_fast(v1[e]); }
    }
    const u32x2 w0 = pack_bf16x4(v0), w1 = pack_bf16x4(v1);
    __builtin_nontemporal_store(u32x4{w0[0], w0[1], w1[0], w1[1]}, (u32x4*)((uint16_t*)g.out + o));
}

// Output rows (and those of the second output and the GELU' input) take vector accesses.
__device__ __forceinline__ bool rows_aligned(const GemmArgs& g)
{
    return ((g.ldo * (g.out_f32 ? 4 : 2)) % 16 == 0) && ((reinterpret_cast<uintptr_t>(g.out) & 15u) == 0) &&
           (!g.preact || (reinterpret_cast<uintptr_t>(g.preact) & 15u) == 0) &&
           (!g.zin || (((reinterpret_cast<uintptr_t>(g.zin) & 7u) == 0) && (g.ldz % 4 == 0)));
}
// dX through GELU' whose pre-activations are fetched ahead of the drain
__device__ __forceinline__ bool drains_dgelu(const GemmArgs& g)
{
    return g.zin && g.dact == TESS_ACT_GELU_ERF && !g.out_f32 && !g.in_f32 && !g.preact && g.act == TESS_ACT_NONE;
}
// bf16 pre-activations of four adjacent columns; zero past the edge
__device__ __forceinline__ u32x2 load_z4(const GemmArgs& g, int row, int col, bool vec)
{
    u32x2 z = {0u, 0u};
    if (row < g.M && col < g.N) {
        const uint16_t* zp = (const uint16_t*)g.zin + (int64_t)row * g.ldz + col;
        if (vec && col + 3 < g.N) {
            z = *(const u32x2*)zp;
        } else {
            for (int e = 0; e < 4; ++e)
                if (col + e < g.N) z[e >> 1] |= (uint32_t)zp[e] << (16 * (e & 1));
        }
    }
    return z;
}
// Calls `body` with the drain mode of this call (all but MODE_BF16_DGELU).
template <typename F>
__device__ __forceinline__ void with_drain_mode(const GemmArgs& g, F&& body)
{
    const bool generic = g.zin || g.act == TESS_ACT_GELU_TANH || (g.out_f32 && (g.act != TESS_ACT_NONE || g.preact)) ||
                         (g.preact && g.act != TESS_ACT_GELU_ERF);
    if (generic) body(std::integral_constant<int, MODE_GENERIC>{});
    else if (g.preact) body(std::integral_constant<int, MODE_BF16_GELU_PRE>{});
    else if (g.out_f32 && g.accumulate) body(std::integral_constant<int, MODE_F32_ACC>{});
    else if (g.out_f32) body(std::integral_constant<int, MODE_F32>{});
    else if (g.act == TESS_ACT_GELU_ERF) body(std::integral_constant<int, MODE_BF16_GELU>{});
    else body(std::integral_constant<int, MODE_BF16>{});
}

}  // namespace tess
