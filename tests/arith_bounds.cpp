// The digit sums of the fused giant steps (fa_arith.h: add_digit) at the edge of their
// bounds, on the CPU: tests/test_arith_bounds.py compiles this file with a stand-in for
// the HIP header and feeds primes on stdin.  For each prime it looks for the products
// of largest magnitude among row-pass words (within 2.65 q) and key words, all of one
// sign, and adds them up as the kernel does; the sums must be the exact ones modulo q
// (128-bit integers).  Prints "ok q" per prime, or the first sum that is off.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "fa_arith.h"

using i128 = __int128;

struct Pair {
  double x, k, r;  // r: what mul returns
};

static long long mod(i128 v, long long q) {
  const long long r = (long long)(v % q);
  return r < 0 ? r + q : r;
}

template <int DNUM>
static bool sums(const std::vector<Pair>& pos, const std::vector<Pair>& neg, double q, double qinv,
                 std::mt19937_64& g) {
  constexpr int R = 16;
  const double start = 0.5 * (q - 1.0);  // a reduced word
  for (int trial = 0; trial < 200; ++trial) {
    double s0[R], s1[R];
    i128 e0[R], e1[R];
    for (int j = 0; j < R; ++j) {
      s0[j] = start;
      s1[j] = -start;
      e0[j] = (i128)start;
      e1[j] = -(i128)start;
    }
    for (int i = 0; i < DNUM; ++i) {
      // the first sum takes the largest products, the second the smallest
      double x0[R], x1[R], k0[R], k1[R], unused[R] = {};
      for (int j = 0; j < R; ++j) {
        const Pair &p = pos[g() % pos.size()], &m = neg[g() % neg.size()];
        x0[j] = p.x;
        k0[j] = p.k;
        x1[j] = m.x;
        k1[j] = m.k;
        e0[j] += (i128)p.x * (i128)p.k;
        e1[j] += (i128)m.x * (i128)m.k;
      }
      add_digit<DNUM>(s0, unused, x0, k0, k0, 1, i, q, qinv);
      std::fill(unused, unused + R, 0.0);
      add_digit<DNUM>(unused, s1, x1, k1, k1, 1, i, q, qinv);
    }
    for (int j = 0; j < R; ++j) {
      // the term of c0 and P, two canonical words
      const double a = q - 1.0 - (double)(g() % 1000), b = q - 1.0 - (double)(g() % 1000);
      s0[j] += mul(a, b, q, qinv);
      e0[j] += (i128)a * (i128)b;
      for (int h = 0; h < 2; ++h) {
        const double got = canon_full(h ? s1[j] : s0[j], q, qinv);
        const long long want = mod(h ? e1[j] : e0[j], (long long)q);
        if ((long long)got != want) {
          std::printf("q %.0f, %d digits: sum %.0f (%.3f q) gives %.0f, exact %lld\n", q, DNUM, h ? s1[j] : s0[j],
                      (h ? s1[j] : s0[j]) / q, got, want);
          return false;
        }
      }
    }
  }
  return true;
}

int main() {
  unsigned long long qq;
  std::mt19937_64 g(11);
  while (std::scanf("%llu", &qq) == 1) {
    const double q = (double)qq, qinv = 1.0 / q, lim = std::floor(2.65 * q);
    std::vector<Pair> all;
    for (int i = 0; i < 300000; ++i) {
      const double x = lim - std::floor((double)(g() >> 11) * 0x1p-53 * 0.02 * lim);
      const double k = q - 1.0 - std::floor((double)(g() >> 11) * 0x1p-53 * 0.02 * q);
      const double sx = i & 1 ? -x : x;
      all.push_back({sx, k, mul(sx, k, q, qinv)});
    }
    std::sort(all.begin(), all.end(), [](const Pair& a, const Pair& b) { return a.r < b.r; });
    const std::vector<Pair> neg(all.begin(), all.begin() + 64), pos(all.end() - 64, all.end());
    if (!(sums<1>(pos, neg, q, qinv, g) && sums<2>(pos, neg, q, qinv, g) && sums<3>(pos, neg, q, qinv, g) &&
          sums<4>(pos, neg, q, qinv, g) && sums<5>(pos, neg, q, qinv, g) && sums<6>(pos, neg, q, qinv, g) &&
          sums<7>(pos, neg, q, qinv, g) && sums<8>(pos, neg, q, qinv, g)))
      return 1;
    std::printf("ok %llu\n", qq);
  }
  return 0;
}
