// Softmax arithmetic of the fp32 attention kernels, shared by chunk prefill and decode, and sums over lane groups.  What an fp32 caller gets is as
// close to the exact result as sums of 32 bits allow: exponents are formed in two floats, sums of products run in short
// chains that meet pairwise (in the kernels), quotients are rounded once.
#pragma once

#include <hip/hip_runtime.h>

namespace sv {

// e^(d / sqrt(D)) of a difference of raw scores (d <= 0, or -infinity).  The exponent d * log2(e) / sqrt(D) is formed in
// two floats, the product and its rounding error with the rest of the constant, and the second one's factor
// 2^lo = 1 + lo * ln 2 applied afterwards: rounded to one float, an exponent of -10 puts the weight off by 3e-7.
// rest: what the score's last addition rounded off, for the low part.
template <int D>
__device__ __forceinline__ float exp_scaled(float d, float rest = 0.f) {
  constexpr double c = 1.4426950408889634074 * (D == 128 ? 0.088388347648318440550 : 0.125);   // log2(e) / sqrt(D)
  constexpr float ch = (float)c, cl = (float)(c - (double)ch);
  const float hi = d * ch;
  // (of -infinity the low part is no number, and the minimum then 1: the weight stays 0.  A d that is no number makes hi,
  // and with it the weight, none either.)
  const float lo = fminf(fmaf(rest, ch, fmaf(d, cl, fmaf(d, ch, -hi))) * 0.69314718f, 1.0f);
  const float p = __builtin_amdgcn_exp2f(hi);
  return fmaf(p, lo, p);
}

// x / l with inv = 1 / l at hand: the product's remainder corrects it, so that the result is rounded once.  (An infinite x has
// none: it stays.)
__device__ __forceinline__ float quotient(float x, float l, float inv) {
  const float r = x * inv, rest = fmaf(-r, l, x);
  return rest == rest ? fmaf(rest, inv, r) : r;
}

// Sum of N registers, pairwise.
template <int N, typename V>
__device__ __forceinline__ float sum_of(const V& v, int at = 0) {
  if constexpr (N == 1) return v[at];
  else return sum_of<N / 2>(v, at) + sum_of<N / 2>(v, at + N / 2);
}

// What a + b, rounded to sum, leaves.
template <typename V>
__device__ __forceinline__ V rest_of(const V& a, const V& b, const V& sum) {
  const V b2 = sum - a;
  return (a - (sum - b2)) + (b - b2);
}

// max / sum over the four lane groups l, l ^ 16, l ^ 32, l ^ 48: two row swaps on the vector ALU (through LDS, as
// ds_bpermute, each step is a round trip of some 100 cycles)
__device__ __forceinline__ void swap16(float x, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float x, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]), b = __uint_as_float(r[1]);
}
__device__ __forceinline__ float groups_max(float x) {
  float a, b;
  swap16(x, a, b);
  swap32(fmaxf(a, b), a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float groups_sum(float x) {
  float a, b;
  swap16(x, a, b);
  swap32(a + b, a, b);
  return a + b;
}

// A running sum in two floats: what an addition rounds off goes into the second one.
struct Sum {
  float hi = 0.f, lo = 0.f;
  __device__ __forceinline__ void scale(float x) { hi *= x, lo *= x; }
  __device__ __forceinline__ void add(float x) {
    const float t = hi + x;
    lo += rest_of(hi, x, t);
    hi = t;
  }
  __device__ __forceinline__ float value() const { return hi + lo; }
};

}  // namespace sv
