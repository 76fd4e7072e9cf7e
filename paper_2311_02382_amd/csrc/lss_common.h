// Device-side building blocks shared by the segment-attention kernels (gfx950).
//
// Matrix-core tile used throughout: V_MFMA_F32_32X32X16_BF16 (single precision: six of them on
// three-part operands, lss_f32.hip).  One wavefront of 64 lanes computes a 32x32 fp32 tile
// C += A(32x16) * B(16x32):
//   lane l holds, for A, row (l % 32), and for B, column (l % 32); both hold the 8
//   contraction slots of half (l / 32);
//   C is 16 floats per lane: element v is row 8*(v/4) + 4*(l/32) + (v%4), column l%32.
// A "fragment" below is one lane's 8 contraction slots.  Which contraction index a
// slot carries is free as long as A and B agree, which the kernels use to feed a C
// tile straight back in as a B operand: slots 8*s..8*s+7 of a C tile (s = 0, 1)
// carry rows 16*s + 8*(e/4) + 4*(l/32) + (e%4), e = 0..7.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lss {

typedef __bf16 bf16_t;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

template <typename T> struct Frag;
template <> struct Frag<bf16_t> { bf16x8 v; };

// C += A * B on the matrix cores, one 32x32x16 step.
__device__ __forceinline__ f32x16 mma(const Frag<bf16_t> &a, const Frag<bf16_t> &b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
}

// C += A * B, one 16x16x32 step: lane l holds, for A, row (l % 16), for B, column (l % 16), both the 8 contraction
// slots of quarter (l / 16); C is 4 floats per lane, rows 4*(l/16) + v, column l % 16.
__device__ __forceinline__ f32x4 mma16(const Frag<bf16_t> &a, const Frag<bf16_t> &b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v, b.v, c, 0, 0, 0);
}

// 8 consecutive elements, 16-byte aligned
template <typename T> __device__ __forceinline__ Frag<T> load_frag(const T *p);
template <> __device__ __forceinline__ Frag<bf16_t> load_frag<bf16_t>(const bf16_t *p)
{
    Frag<bf16_t> f;
    f.v = *reinterpret_cast<const bf16x8 *>(p);
    return f;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Dropout on the attention weights (Section 2.2), decided per weight from its position in the whole
// sequence, so that a segment drops what the sequential computation would drop there (Section 3,
// Principle 3): the weight of (batch*head bh, global query row, key col) is kept when
//     mix32(row key + column key) >= round(p * 2^32),
// where the row key mixes (low half of the seed, bh, row) and the column key (high half of the seed,
// col); mix32 is a published 32-bit mixing function (xorshift-multiply, two rounds).  No state, no
// stream.  The split into a row and a column key is what a kernel needs: one whose lanes own query
// rows keeps a row key per lane, one whose lanes own keys a column key per lane, and the other key
// of a tile's 64 rows or columns is computed once per tile.
__device__ __forceinline__ uint32_t mix32(uint32_t x)
{
    x = (x ^ (x >> 16)) * 0x7feb352du;
    x = (x ^ (x >> 15)) * 0x846ca68bu;
    return x ^ (x >> 16);
}
__device__ __forceinline__ uint32_t drop_row_key(uint32_t seed_lo, uint32_t bh, uint32_t row)
{
    return mix32(mix32(seed_lo + 0x9e3779b9u * (bh + 1u)) ^ row);
}
// `cs` = drop_col_seed(seed_hi), the same for every column
__device__ __forceinline__ uint32_t drop_col_seed(uint32_t seed_hi) { return mix32(seed_hi + 0x85ebca6bu); }
__device__ __forceinline__ uint32_t drop_col_key(uint32_t cs, uint32_t col) { return mix32(cs ^ col); }
__device__ __forceinline__ bool drop_keep(uint32_t row_key, uint32_t col_key, uint32_t thr)
{
    return mix32(row_key + col_key) >= thr;
}
// ... in three pieces: drop_keep(r, c, thr) = drop_decide(drop_round2(drop_round1(r, c)), thr).  The mixing function's last
// step, x ^ (x >> 16), leaves the upper half of x as it is: the lower half of what is compared matters only where the upper one equals
// thr's, so that x ^ (thr >> 16) compares alike (an xor with a constant takes 3 cycles, one with the shifted value 5).
__device__ __forceinline__ uint32_t drop_round1(uint32_t row_key, uint32_t col_key)
{
    const uint32_t x = row_key + col_key;
    return (x ^ (x >> 16)) * 0x7feb352du;
}
__device__ __forceinline__ uint32_t drop_round2(uint32_t x) { return (x ^ (x >> 15)) * 0x846ca68bu; }
__device__ __forceinline__ bool drop_decide(uint32_t x, uint32_t thr) { return (x ^ (thr >> 16)) >= thr; }

// Exact GeLU, u Phi(u), and its derivative Phi(u) + u phi(u) (Phi, phi: the standard normal's distribution function and
// density).  For u <= 0, Phi(u) = exp(-u^2/2) Q(t) t with t = 1 / (1 + 0.45 |u| / sqrt 2), Q the polynomial of degree 9 that
// makes the largest relative error over t in (0, 1] smallest (3.2e-8; Lawson's iteration against erfcx in 64 bits); Phi(u) =
// 1 - Phi(-u) otherwise.  Through erff, whose both halves nearly every wavefront runs, GeLU took 39 vector instructions per
// element and its kernel was bound by them; 20 here.  In fp32, against 64 bits: GeLU of Gaussian values 3.7e-8 of their norm
// either way; Phi of values down to -5 1.4e-6 of itself, where 1 + erf had cancelled to 4.9e-2.
__device__ __forceinline__ float gelu_phi(float u, float &e)        // e: exp(-u^2/2)
{
    const float t = __builtin_amdgcn_rcpf(fmaf(fabsf(u), 0.31819805153394637f, 1.0f));
    float q = -0.020695484f;
    q = fmaf(q, t, 0.0953436f);
    q = fmaf(q, t, -0.15029061f);
    q = fmaf(q, t, 0.07119989f);
    q = fmaf(q, t, -0.011178641f);
    q = fmaf(q, t, 0.05997511f);
    q = fmaf(q, t, 0.087626085f);
    q = fmaf(q, t, 0.11413582f);
    q = fmaf(q, t, 0.12694158f);
    q = fmaf(q, t, 0.12694266f);
    e = fast_exp2(u * u * -0.72134752044448170f);
    const float tail = q * t * e;
    return u < 0.f ? tail : 1.0f - tail;
}
__device__ __forceinline__ float gelu_value(float u)
{
    float e;
    return u * gelu_phi(u, e);
}
__device__ __forceinline__ float gelu_slope(float u)
{
    float e;
    const float phi = gelu_phi(u, e);
    return fmaf(u * 0.3989422804014327f, e, phi);
}

} // namespace lss
