// Activations of Eq. (1) and the FP32 MFMA step shared by the MLP kernels
// (the fused two-hidden-layer kernels and the layer-by-layer path).
#pragma once

#include <math.h>

#include "common.h"

namespace nnp {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float act_f(int code, float z) {
  switch (code) {
    case NN_ACT_GAUSSIAN: return __builtin_amdgcn_exp2f(-1.4426950408889634f * z * z);
    case NN_ACT_RELU: return z > 0.f ? z : 0.f;
    case NN_ACT_TANH: return tanhf(z);
    default: return z;
  }
}
__device__ __forceinline__ float act_d(int code, float z, float a) {
  switch (code) {
    case NN_ACT_GAUSSIAN: return -2.0f * z * a;
    case NN_ACT_RELU: return z > 0.f ? 1.f : 0.f;
    case NN_ACT_TANH: return 1.0f - a * a;
    default: return 1.0f;
  }
}

__device__ __forceinline__ float act_d2(int code, float z, float a) {
  switch (code) {
    case NN_ACT_GAUSSIAN: return fmaf(4.0f * z, z, -2.0f) * a;
    case NN_ACT_TANH: return -2.0f * a * (1.0f - a * a);
    default: return 0.0f;
  }
}

// act(z + bias) and its derivative for four z, one branch for all of them.  With
// PASS_NAN, ReLU of NaN is NaN too, not zero.
template <bool PASS_NAN>
__device__ __forceinline__ void act4(int code, const floatx4& z, float bias, float (&a)[4], float (&d)[4]) {
  auto each = [&](int c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float x = z[j] + bias;
      a[j] = act_f(c, x);
      if (PASS_NAN && c == NN_ACT_RELU) a[j] = x != x ? x : a[j];
      d[j] = act_d(c, x, a[j]);
    }
  };
  switch (code) {
    case NN_ACT_GAUSSIAN: each(NN_ACT_GAUSSIAN); break;
    case NN_ACT_RELU: each(NN_ACT_RELU); break;
    case NN_ACT_TANH: each(NN_ACT_TANH); break;
    default: each(NN_ACT_LINEAR); break;
  }
}

// FP32 products use v_mfma_f32_16x16x4_f32 over 16-wide k blocks: lane
// (lm, lk) holds the four k values kb + 4 lk + i (i = 0..3) of its A row and
// B column, and the i-th of four MFMAs takes element i.  The four MFMAs
// together cover the whole block (each product a_k b_k once), so every lane
// fetches its operands as one 16-byte vector.
__device__ __forceinline__ float4 ld4(const float* p, int k, int kmax, bool vec) {
  if (vec && k + 3 < kmax) return *reinterpret_cast<const float4*>(p + k);
  float4 v;
  v.x = k < kmax ? p[k] : 0.f;
  v.y = k + 1 < kmax ? p[k + 1] : 0.f;
  v.z = k + 2 < kmax ? p[k + 2] : 0.f;
  v.w = k + 3 < kmax ? p[k + 3] : 0.f;
  return v;
}

__device__ __forceinline__ floatx4 mma4_f32(floatx4 acc, const float4& a, const float4& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc, 0, 0, 0);
}

// Products in the MLP run in one of three modes:
//   kFp32  - FP32 operands, v_mfma_f32_16x16x4_f32;
//   kBf16  - operands rounded to BF16, v_mfma_f32_16x16x32_bf16, FP32 sums;
//   kBf16x3 - each operand split x = hi + lo with hi, lo in BF16 and the
//            product taken as hi*hi + hi*lo + lo*hi (three BF16 MFMAs, FP32
//            sums): about 16 significant bits per operand.
enum { kFp32 = 0, kBf16 = 1, kBf16x3 = 2 };

__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const __bf16 h = (__bf16)x[q];
    hi[q] = h;
    lo[q] = (__bf16)(x[q] - (float)h);
  }
}

// An FP32 value as three BF16 parts, x = h + m + l (the splitting of a long
// significand into shorter ones that error-free products use): each part rounds
// what the one before left, and 3 x 8 bits hold all 24.  Infinities, NaN and
// values beyond the largest BF16 one have no such parts: m or l, and with it
// every sum they enter, is then infinite or not a number, which the caller looks
// for.  Below about 1e-33 the low parts are subnormal and the bits beyond them
// are lost.
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
struct Split3 {
  bf16x8 h, m, l;
};
__device__ __forceinline__ void split_operand(const float (&x)[8], Split3& p) {
  auto pack = [](float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
  };
  auto low = [](uint32_t p) { return __uint_as_float(p << 16); };
  auto high = [](uint32_t p) { return __uint_as_float(p & 0xffff0000u); };
  u32x4v vh, vm, vl;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float x0 = x[2 * q], x1 = x[2 * q + 1];
    vh[q] = pack(x0, x1);
    const float r0 = x0 - low(vh[q]), r1 = x1 - high(vh[q]);
    vm[q] = pack(r0, r1);
    vl[q] = pack(r0 - low(vm[q]), r1 - high(vm[q]));
  }
  p.h = __builtin_bit_cast(bf16x8, vh);
  p.m = __builtin_bit_cast(bf16x8, vm);
  p.l = __builtin_bit_cast(bf16x8, vl);
}

// The same eight values as they are, for products by FP32 instructions.
struct Whole {
  float4 lo, hi;
};
__device__ __forceinline__ void split_operand(const float (&x)[8], Whole& p) {
  p.lo = make_float4(x[0], x[1], x[2], x[3]);
  p.hi = make_float4(x[4], x[5], x[6], x[7]);
}

// acc[g] += a b[g] for products of values in three parts: the six partial
// products down to 2^-16 of the whole, the small ones first (what is left
// out, m l + l m + l l, is below 2^-23 of a product and of either sign).
template <int G>
__device__ __forceinline__ void mma_parts(floatx4* acc, const Split3& a, const Split3 (&b)[G]) {
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b[g].h, acc[g], 0, 0, 0);
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b[g].l, acc[g], 0, 0, 0);
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.m, b[g].m, acc[g], 0, 0, 0);
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.m, b[g].h, acc[g], 0, 0, 0);
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b[g].m, acc[g], 0, 0, 0);
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b[g].h, acc[g], 0, 0, 0);
}
// acc[g] += a b[g] by FP32 instructions (lane (lm, lk) holds the k values
// 8 lk + i of both operands).
template <int G>
__device__ __forceinline__ void mma_parts(floatx4* acc, const Whole& a, const Whole (&b)[G]) {
#pragma unroll
  for (int g = 0; g < G; ++g) acc[g] = mma4_f32(mma4_f32(acc[g], a.lo, b[g].lo), a.hi, b[g].hi);
}

template <int MODE>
__device__ __forceinline__ floatx4 mma_bf16(floatx4 acc, const bf16x8& ah, const bf16x8& al, const bf16x8& bh,
                                            const bf16x8& bl) {
  if constexpr (MODE == kBf16x3) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, acc, 0, 0, 0);
  }
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, acc, 0, 0, 0);
}

}  // namespace nnp
