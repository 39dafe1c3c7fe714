// Device arithmetic shared by the kernel files: exact float64 residues (see the
// header of fa_kernels.hip for the bounds) and the automorphism's permutation.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

__device__ __forceinline__ double reduce(double x, double q, double qinv) {
  return __fma_rn(-rint(x * qinv), q, x);
}
__device__ __forceinline__ double mulc(double a, double w, double wp, double q) {
  const double h = a * w;
  const double l = __fma_rn(a, w, -h);
  const double t = rint(a * wp);
  return __fma_rn(-t, q, h) + l;
}
__device__ __forceinline__ double mul(double a, double b, double q, double qinv) {
  const double h = a * b;
  const double l = __fma_rn(a, b, -h);
  const double t = rint(h * qinv);
  return __fma_rn(-t, q, h) + l;
}
// x in (-q, 2q) -> [0, q)
__device__ __forceinline__ double canon(double x, double q) {
  x = x < 0.0 ? x + q : x;
  return x >= q ? x - q : x;
}
// full canonical reduction of |x| < 2^52
__device__ __forceinline__ double canon_full(double x, double q, double qinv) {
  x = reduce(x, q, qinv);
  return x < 0.0 ? x + q : x;
}

// A key-switch sum over words that come straight from a row pass (within 2.66 q, see
// ct_bfly in fa_kernels.hip; a product with a canonical word is then within
// 0.5 + 0.375 * 2.66): from a reduced word it takes kSumDigits of them and one
// product of two canonical words before it could leave 8 q and 2^53, above which
// integers are no longer exact.
constexpr int kSumDigits = 4, kMaxDigits = 8;
constexpr double kRowWord = 2.66;
static_assert(0.5 + kSumDigits * (0.5 + 0.375 * kRowWord) + 0.75 < 8.0, "a sum stays exact");
static_assert(2 * kSumDigits >= kMaxDigits, "one reduction among the digits is enough");
// Digit i of DNUM of both polynomials' sums: s_h[j] += x[j] key_h[stride j].
template <int DNUM, int R>
__device__ __forceinline__ void add_digit(double (&s0)[R], double (&s1)[R], const double (&x)[R],
                                          const double* __restrict__ key0, const double* __restrict__ key1, int stride,
                                          int i, double q, double qinv) {
  static_assert(DNUM <= kMaxDigits, "see kSumDigits");
  if (DNUM > kSumDigits && i == kSumDigits) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      s0[j] = reduce(s0[j], q, qinv);
      s1[j] = reduce(s1[j], q, qinv);
    }
  }
#pragma unroll
  for (int j = 0; j < R; ++j) {
    s0[j] += mul(x[j], key0[stride * j], q, qinv);
    s1[j] += mul(x[j], key1[stride * j], q, qinv);
  }
}

// Index permutation of the Galois automorphism X -> X^gal in NTT order:
// output slot i of the forward transform holds a(psi^(2 brev(i) + 1)), so
// sigma(a)^[i] = a^[pi(i)] with 2 brev(pi(i)) + 1 = gal (2 brev(i) + 1) mod 2N.
__device__ __forceinline__ uint32_t perm(uint32_t i, uint32_t gal, int logn) {
  const uint32_t e = 2u * (__brev(i) >> (32 - logn)) + 1u;
  const uint32_t e2 = (gal * e) & ((2u << logn) - 1u);
  return __brev((e2 - 1u) >> 1) >> (32 - logn);
}

}  // namespace
