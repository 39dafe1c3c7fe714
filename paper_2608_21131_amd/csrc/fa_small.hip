// Kernels of small rings (N <= 2^FA_SMALL_LOGN): one limb fits a workgroup's LDS.
//
// A ring this small leaves the two-pass kernels of fa_kernels.hip waiting on
// launches: a rotation at N = 2^13 with 3+1 primes was seven of them, 2-12 us
// each, for 0.05 us of HBM traffic.  Here a workgroup of N/16 threads keeps a
// whole limb in registers (16 words a thread) and exchanges through LDS once
// per three or four stages, so the transforms never go through HBM between
// passes, and the key products run in the same kernels:
//   k_sr_inv      inverse transform and scaling of c1's limbs,
//   k_sr_modup    conversion of a digit to one prime and its forward transform,
//   k_sr_ksinv    key-switch sum on a special prime and its inverse transform,
//   k_sr_finish   conversion to one ciphertext prime, forward transform, the
//                 key-switch sum on that prime, ModDown and the additions.
// With one special prime (one limb per digit) the first runs inside the second
// and the third's inverse inside the fourth when there are workgroups to spare
// (FUSED), its sums formed before by k_sr_special: a rotation is three launches,
// otherwise four.  Measured: a rotation at N = 2^13, 3+1 primes 43.5 -> 31.0 us,
// the 7-step row fold 340 -> 227 us, twenty-four calls of all kinds at N = 2^11 to
// 2^13 1.9 times as fast on average.  What is left of a rotation: the inverse
// transform on one CU (4.8 us, twice: 7.7k clocks of issue and 4k of LDS), the
// quarter's share of the forward one, and 2-3 us a launch.
//
// Bounds (in units of q, see fa_kernels.hip for the products): fwd_reduces()
// and inv_reduces() place the reductions stage by stage so that a product's
// operand stays within 8q, where it is exact.

#include <algorithm>
#include <type_traits>

#include "fa_arith.h"
#include "fa_internal.h"

namespace {

template <int LOGN>
struct Ring {
  static constexpr int N = 1 << LOGN;
  static constexpr int T = N / 16;       // threads per limb, 16 words each
  static constexpr int LDS = N + N / 8;  // one pad word per 8: see pad()
};
// LDS position of word i: with one pad word per 8 both the strided reads (64
// lanes on a block of 8..64 words each) and the reads of 8 or 16 consecutive
// words per lane spread over the banks
__device__ __forceinline__ int pad(int i) { return i + (i >> 3); }

// stages of pass p: 4, then 4s and 3s to log2 N
constexpr int pass_stages(int logn, int p) {
  const int plan[4][4] = {{4, 3, 3, 0}, {4, 4, 3, 0}, {4, 4, 4, 0}, {4, 3, 3, 3}};
  return plan[logn - 10][p];
}
constexpr int pass_first(int logn, int p) { return p == 0 ? 0 : pass_first(logn, p - 1) + pass_stages(logn, p - 1); }
constexpr int pass_count(int logn) { return logn > 12 ? 4 : 3; }

// Does forward stage s reduce its first operand?  From c <= 1 a lazy stage
// leaves 1.375 c + 0.5 and a reducing one 1 + 0.375 c; a stage reduces when the
// lazy bound would pass 7.5 (the outputs then stay below 7.5 q, the epilogue's
// difference with a reduced word below 8 q).
constexpr bool fwd_reduces(int s) {
  double c = 1.0;
  for (int i = 0;; ++i) {
    const bool r = 1.375 * c + 0.5 > 7.5;
    if (i == s) return r;
    c = r ? 1.0 + 0.375 * c : 1.375 * c + 0.5;
  }
}
// Does the k-th inverse stage (from the last) reduce its sum?  Inputs within c
// give sums within 2c and products within 0.5 + 0.75 c; inputs stay within 4.
constexpr bool inv_reduces(int k) {
  double c = 1.0;
  for (int i = 0;; ++i) {
    const bool r = 2.0 * c > 4.0;
    if (i == k) return r;
    const double y = 0.5 + 0.75 * c, x = r ? 0.5 : 2.0 * c;
    c = x > y ? x : y;
  }
}

// word of group v, element m in the pass of R stages from stage S
template <int LOGN, int S, int R>
__device__ __forceinline__ int word(int v, int m) {
  constexpr int ls = LOGN - S - R;
  const int u = (int)threadIdx.x + Ring<LOGN>::T * v;
  return ((u >> ls) << (ls + R)) + (u & ((1 << ls) - 1)) + (m << ls);
}

// A thread's twiddles of the passes after the first, 14 or 15 words a pass,
// loaded before the data they meet: a pass starts behind a barrier, and waiting
// there for its twiddles (L2 or further) took longer than its arithmetic.
// Group v of the pass holds stage s1's 2^s1 words at v (E - 1) + 2^s1 - 1.
// PRE false (launches that fill the chip): read where they are used; the
// registers saved let two workgroups share a CU, which hides as much.
// The largest of either kind spill: k_sr_ksinv at N = 2^13 4 registers of 256 (PRE),
// k_sr_modup at N = 2^10 with two primes a digit 8 of 128.
template <int LOGN, bool PRE>
struct Twiddles {
  double w[PRE ? pass_count(LOGN) - 1 : 1][PRE ? 15 : 1];
};
template <int LOGN, bool PRE, int P = 1>
__device__ __forceinline__ void load_twiddles(Twiddles<LOGN, PRE>& tw, const double* __restrict__ w) {
  if constexpr (!PRE) return;
  constexpr int S = pass_first(LOGN, P), R = pass_stages(LOGN, P), ls = LOGN - S - R, E = 1 << R;
#pragma unroll
  for (int v = 0; v < 16 / E; ++v) {
    const int blk = ((int)threadIdx.x + Ring<LOGN>::T * v) >> ls;
#pragma unroll
    for (int s1 = 0; s1 < R; ++s1)
#pragma unroll
      for (int i = 0; i < (1 << s1); ++i)
        if constexpr (PRE) tw.w[P - 1][v * (E - 1) + (1 << s1) - 1 + i] = w[(1 << (S + s1)) + (blk << s1) + i];
  }
  if constexpr (PRE && P + 1 < pass_count(LOGN)) load_twiddles<LOGN, PRE, P + 1>(tw, w);
}
// w: the table of the prime (the first pass's twiddles are the same for all threads)
template <int LOGN, int P, bool PRE>
__device__ __forceinline__ double twiddle(const Twiddles<LOGN, PRE>& tw, const double* __restrict__ w, int v, int s1,
                                          int i) {
  constexpr int S = pass_first(LOGN, P), R = pass_stages(LOGN, P), E = 1 << R;
  if constexpr (P == 0) return w[(1 << s1) + i];
  else if constexpr (!PRE)
    return w[(1 << (S + s1)) + ((((int)threadIdx.x + Ring<LOGN>::T * v) >> (LOGN - S - R)) << s1) + i];
  else return tw.w[P - 1][v * (E - 1) + (1 << s1) - 1 + i];
}

template <int LOGN, int P, bool PRE>
__device__ __forceinline__ void fwd_pass(double (&x)[16], const Twiddles<LOGN, PRE>& tw,
                                         const double* __restrict__ w, double q, double qinv) {
  constexpr int S = pass_first(LOGN, P), R = pass_stages(LOGN, P), E = 1 << R;
#pragma unroll
  for (int s1 = 0; s1 < R; ++s1) {
    const int half = E >> (s1 + 1);
#pragma unroll
    for (int v = 0; v < 16 / E; ++v)
#pragma unroll
      for (int m = 0; m < E; ++m) {
        if (m & half) continue;
        double& a = x[v * E + m];
        double& b = x[v * E + m + half];
        const double u = fwd_reduces(S + s1) ? reduce(a, q, qinv) : a;
        const double t = mul(b, twiddle<LOGN, P, PRE>(tw, w, v, s1, m >> (R - s1)), q, qinv);
        a = u + t;
        b = u - t;
      }
  }
}
template <int LOGN, int P, bool PRE>
__device__ __forceinline__ void inv_pass(double (&x)[16], const Twiddles<LOGN, PRE>& tw,
                                         const double* __restrict__ w, double q, double qinv) {
  constexpr int S = pass_first(LOGN, P), R = pass_stages(LOGN, P), E = 1 << R;
#pragma unroll
  for (int s1 = R - 1; s1 >= 0; --s1) {
    const int half = E >> (s1 + 1);
#pragma unroll
    for (int v = 0; v < 16 / E; ++v)
#pragma unroll
      for (int m = 0; m < E; ++m) {
        if (m & half) continue;
        double& a = x[v * E + m];
        double& b = x[v * E + m + half];
        const double u = a + b, d = a - b;
        a = inv_reduces(LOGN - 1 - S - s1) ? reduce(u, q, qinv) : u;
        b = mul(d, twiddle<LOGN, P, PRE>(tw, w, v, s1, m >> (R - s1)), q, qinv);
      }
  }
}
// registers <-> LDS in a pass's own layout.  A thread writes back exactly the
// words it read, so one barrier per exchange is enough.
template <int LOGN, int S, int R>
__device__ __forceinline__ void put(const double (&x)[16], double* sm) {
#pragma unroll
  for (int v = 0; v < (16 >> R); ++v)
#pragma unroll
    for (int m = 0; m < (1 << R); ++m) sm[pad(word<LOGN, S, R>(v, m))] = x[(v << R) + m];
}
template <int LOGN, int S, int R>
__device__ __forceinline__ void get(double (&x)[16], const double* sm) {
#pragma unroll
  for (int v = 0; v < (16 >> R); ++v)
#pragma unroll
    for (int m = 0; m < (1 << R); ++m) x[(v << R) + m] = sm[pad(word<LOGN, S, R>(v, m))];
}

// Forward transform of x (word tid + T m at x[m], |x| <= q) into sm (padded,
// transform order, within 7.5 q); synchronised on return.
template <int LOGN, bool PRE, int P = 0>
__device__ __forceinline__ void fwd_limb(double (&x)[16], const Twiddles<LOGN, PRE>& tw,
                                         const double* __restrict__ w, double q, double qinv, double* sm) {
  constexpr int S = pass_first(LOGN, P), R = pass_stages(LOGN, P);
  if constexpr (P > 0) get<LOGN, S, R>(x, sm);
  fwd_pass<LOGN, P, PRE>(x, tw, w, q, qinv);
  put<LOGN, S, R>(x, sm);
  __syncthreads();
  if constexpr (P + 1 < pass_count(LOGN)) fwd_limb<LOGN, PRE, P + 1>(x, tw, w, q, qinv, sm);
}
// Inverse transform of x (transform order, word tid + T m at x[m], |x| <= q) to
// natural order, word tid + T m at x[m], within 4 q and not yet scaled.  The
// first exchange takes the coalesced words to the last pass's runs of 8 or 16.
// A thread last reads exactly the words of sm that fwd_limb writes first.
template <int LOGN, bool PRE, int P = pass_count(LOGN)>
__device__ __forceinline__ void inv_limb(double (&x)[16], const Twiddles<LOGN, PRE>& tw,
                                         const double* __restrict__ w, double q, double qinv, double* sm) {
  if constexpr (P == pass_count(LOGN)) {
    put<LOGN, 0, 4>(x, sm);
  } else {
    inv_pass<LOGN, P, PRE>(x, tw, w, q, qinv);
    if constexpr (P > 0) put<LOGN, pass_first(LOGN, P), pass_stages(LOGN, P)>(x, sm);
  }
  if constexpr (P > 0) {
    __syncthreads();
    get<LOGN, pass_first(LOGN, P - 1), pass_stages(LOGN, P - 1)>(x, sm);
    inv_limb<LOGN, PRE, P - 1>(x, tw, w, q, qinv, sm);
  }
}
// Forward transform by parts: one of the 2^LP = 4 contiguous quarters of the
// output.  The first two stages are formed for the quarter alone (three products
// for its word of every four instead of one a word), the other LOGN - 2 run on
// N/4 words: 4 a thread for two stages, then 8 words on half the threads.  A
// single limb's transform is bound by one CU's issue and LDS rates (4.8 us at
// N = 2^13); the quarter takes about a third of that.
constexpr int kParts = 4;
constexpr int part_stages(int logn, int p) {
  const int plan[4][3] = {{3, 3, 0}, {3, 2, 2}, {3, 3, 2}, {3, 3, 3}};
  return plan[logn - 10][p];
}
constexpr int part_first(int logn, int p) { return p == 0 ? 4 : part_first(logn, p - 1) + part_stages(logn, p - 1); }
constexpr int part_passes(int logn) { return logn == 10 ? 2 : 3; }
template <int LOGN>
struct PartTwiddles {
  double w[part_passes(LOGN)][7];
};
template <int LOGN, int P = 0>
__device__ __forceinline__ void load_part_twiddles(PartTwiddles<LOGN>& tw, const double* __restrict__ w, int part) {
  constexpr int S = part_first(LOGN, P), R = part_stages(LOGN, P), ls = LOGN - S - R, E = 1 << R;
  constexpr int T2 = Ring<LOGN>::T / 2;
  const int tid = threadIdx.x & (T2 - 1);
#pragma unroll
  for (int v = 0; v < 8 / E; ++v) {
    const int blk = (part << (S - 2)) + ((tid + T2 * v) >> ls);
#pragma unroll
    for (int s1 = 0; s1 < R; ++s1)
#pragma unroll
      for (int i = 0; i < (1 << s1); ++i)
        tw.w[P][v * (E - 1) + (1 << s1) - 1 + i] = w[(1 << (S + s1)) + (blk << s1) + i];
  }
  if constexpr (P + 1 < part_passes(LOGN)) load_part_twiddles<LOGN, P + 1>(tw, w, part);
}
template <int LOGN, int P = 0>
__device__ __forceinline__ void part_passes_run(const PartTwiddles<LOGN>& tw, double q, double qinv, double* sm) {
  constexpr int S = part_first(LOGN, P), R = part_stages(LOGN, P), ls = LOGN - S - R, E = 1 << R;
  constexpr int T2 = Ring<LOGN>::T / 2;
  const int tid = threadIdx.x;
  if (tid < T2) {
    double x[8];
#pragma unroll
    for (int v = 0; v < 8 / E; ++v)
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int u = tid + T2 * v;
        x[v * E + m] = sm[pad(((u >> ls) << (ls + R)) + (u & ((1 << ls) - 1)) + (m << ls))];
      }
#pragma unroll
    for (int s1 = 0; s1 < R; ++s1) {
      const int half = E >> (s1 + 1);
#pragma unroll
      for (int v = 0; v < 8 / E; ++v)
#pragma unroll
        for (int m = 0; m < E; ++m) {
          if (m & half) continue;
          double& a = x[v * E + m];
          double& b = x[v * E + m + half];
          const double u = fwd_reduces(S + s1) ? reduce(a, q, qinv) : a;
          const double t = mul(b, tw.w[P][v * (E - 1) + (1 << s1) - 1 + (m >> (R - s1))], q, qinv);
          a = u + t;
          b = u - t;
        }
    }
#pragma unroll
    for (int v = 0; v < 8 / E; ++v)
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int u = tid + T2 * v;
        sm[pad(((u >> ls) << (ls + R)) + (u & ((1 << ls) - 1)) + (m << ls))] = x[v * E + m];
      }
  }
  __syncthreads();
  if constexpr (P + 1 < part_passes(LOGN)) part_passes_run<LOGN, P + 1>(tw, q, qinv, sm);
}
// x: the whole limb as for fwd_limb; sm receives the quarter's N/4 words
template <int LOGN>
__device__ __forceinline__ void fwd_part(const double (&x)[16], const PartTwiddles<LOGN>& tw,
                                         const double* __restrict__ w, int part, double q, double qinv, double* sm) {
  static_assert(!fwd_reduces(0) && !fwd_reduces(1), "the first two stages are lazy");
  using G = Ring<LOGN>;
  const int p1 = part >> 1;
  const double w0 = w[1], w1 = w[2 + p1], w2 = w[4 + part], w3 = w[8 + 2 * part], w4 = w[9 + 2 * part];
  const double s0 = p1 ? -1.0 : 1.0, s1 = part & 1 ? -1.0 : 1.0;
  double y[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const double u0 = x[m] + s0 * mul(x[m + 8], w0, q, qinv);
    const double u1 = x[m + 4] + s0 * mul(x[m + 12], w0, q, qinv);
    y[m] = u0 + s1 * mul(u1, w1, q, qinv);
  }
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const double u = fwd_reduces(2) ? reduce(y[m], q, qinv) : y[m];
    const double t = mul(y[m + 2], w2, q, qinv);
    y[m] = u + t;
    y[m + 2] = u - t;
  }
#pragma unroll
  for (int m = 0; m < 4; m += 2) {
    const double u = fwd_reduces(3) ? reduce(y[m], q, qinv) : y[m];
    const double t = mul(y[m + 1], m ? w4 : w3, q, qinv);
    y[m] = u + t;
    y[m + 1] = u - t;
  }
  __syncthreads();  // an inverse transform before this one has been read out of sm
#pragma unroll
  for (int m = 0; m < 4; ++m) sm[pad(threadIdx.x + G::T * m)] = y[m];
  __syncthreads();
  part_passes_run<LOGN>(tw, q, qinv, sm);
}
// A workgroup's share of a forward transform: whole limbs or quarters (PARTS)
template <int LOGN, bool PARTS, bool PRE>
struct Fwd {
  static constexpr int WORDS = PARTS ? 4 : 16;  // output words a thread, base + tid + T m
  std::conditional_t<PARTS, PartTwiddles<LOGN>, Twiddles<LOGN, PRE>> tw;
  const double* __restrict__ w;
  int part;
  __device__ int base() const { return PARTS ? part << (LOGN - 2) : 0; }
  __device__ void load(const double* __restrict__ table, int p) {
    w = table;
    part = p;
    if constexpr (PARTS) load_part_twiddles<LOGN>(tw, w, part);
    else load_twiddles<LOGN, PRE>(tw, w);
  }
  __device__ void run(double (&x)[16], double q, double qinv, double* sm) const {
    if constexpr (PARTS) fwd_part<LOGN>(x, tw, w, part, q, qinv, sm);
    else fwd_limb<LOGN, PRE>(x, tw, w, q, qinv, sm);
  }
};
// x[m] = word tid + T m of a limb
template <int LOGN>
__device__ __forceinline__ void load_limb(double (&x)[16], const double* __restrict__ a) {
#pragma unroll
  for (int m = 0; m < 16; ++m) x[m] = a[threadIdx.x + Ring<LOGN>::T * m];
}

// ---------------------------------------------------------------------------
// plain transforms of listed limbs (src -> ptr)
// ---------------------------------------------------------------------------
template <int LOGN>
__global__ __launch_bounds__(Ring<LOGN>::T) void k_sr_fwd_list(LimbList ll, const DevPrime* __restrict__ pr,
                                                               const double* __restrict__ tw) {
  using G = Ring<LOGN>;
  constexpr bool PRE = true;  // at most FA_MAXL workgroups, fewer than CUs
  __shared__ double sm[G::LDS];
  const int pi = ll.prime[blockIdx.x], tid = threadIdx.x;
  const double q = pr[pi].q, qinv = pr[pi].qinv;
  const double* src = ll.src[blockIdx.x];
  double* a = ll.ptr[blockIdx.x];
  const double* __restrict__ w = tw + (size_t)pi * G::N;
  double x[16];
  load_limb<LOGN>(x, src);
  Twiddles<LOGN, PRE> tt;
  load_twiddles<LOGN, PRE>(tt, w);
  fwd_limb<LOGN, PRE>(x, tt, w, q, qinv, sm);
#pragma unroll
  for (int m = 0; m < 16; ++m) a[tid + G::T * m] = canon_full(sm[pad(tid + G::T * m)], q, qinv);
}
template <int LOGN>
__global__ __launch_bounds__(Ring<LOGN>::T) void k_sr_inv_list(LimbList ll, const DevPrime* __restrict__ pr,
                                                               const double* __restrict__ tw) {
  using G = Ring<LOGN>;
  constexpr bool PRE = true;  // at most FA_MAXL workgroups, fewer than CUs
  __shared__ double sm[G::LDS];
  const int pi = ll.prime[blockIdx.x], tid = threadIdx.x;
  const double q = pr[pi].q, qinv = pr[pi].qinv, sc = ll.scale[blockIdx.x], scp = sc * qinv;
  double* a = ll.ptr[blockIdx.x];
  const double* __restrict__ w = tw + (size_t)pi * G::N;
  double x[16];
  load_limb<LOGN>(x, ll.src[blockIdx.x]);
  Twiddles<LOGN, PRE> tt;
  load_twiddles<LOGN, PRE>(tt, w);
  // in place: every word is in registers before inv_limb's first barrier
  inv_limb<LOGN, PRE>(x, tt, w, q, qinv, sm);
#pragma unroll
  for (int m = 0; m < 16; ++m) a[tid + G::T * m] = canon_full(mulc(x[m], sc, scp, q), q, qinv);
}

// ---------------------------------------------------------------------------
// ModUp.  Item b (of an outer and an inner index) reads c1 at
// src + (b / inner) * outer_st + (b % inner) * inner_st and owns
// ext + b * dnum * np * N.  A digit's own limbs of ext are read from c1 by the
// key-switch kernels, so those slots hold the coefficients between k_sr_inv and
// k_sr_modup.
// ---------------------------------------------------------------------------
struct SrUp {
  const double* src;
  double* ext;
  size_t outer_st, inner_st;
  int inner, L, np, alpha, dnum;
};

template <int LOGN, bool PRE>
__global__ __launch_bounds__(Ring<LOGN>::T, PRE ? 1 : 4) void k_sr_inv(SrUp a, const DevPrime* __restrict__ pr,
                                                          const double* __restrict__ twi,
                                                          const double* __restrict__ scale) {
  using G = Ring<LOGN>;
  __shared__ double sm[G::LDS];
  const int t = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const double q = pr[t].q, qinv = pr[t].qinv, sc = scale[t], scp = sc * qinv;
  const double* __restrict__ w = twi + (size_t)t * G::N;
  double x[16];
  load_limb<LOGN>(x, a.src + (b / a.inner) * a.outer_st + (b % a.inner) * a.inner_st + (size_t)t * G::N);
  Twiddles<LOGN, PRE> tt;
  load_twiddles<LOGN, PRE>(tt, w);
  inv_limb<LOGN, PRE>(x, tt, w, q, qinv, sm);
  double* y = a.ext + (((size_t)b * a.dnum + t / a.alpha) * a.np + t) * G::N;
#pragma unroll
  for (int m = 0; m < 16; ++m) y[tid + G::T * m] = canon_full(mulc(x[m], sc, scp, q), q, qinv);
}

// One workgroup per (digit, prime outside it) and part.  FUSED (one limb per
// digit): the digit's inverse transform runs here too, once per workgroup.
template <int LOGN, int ALPHA, bool FUSED, bool PARTS>
__global__ __launch_bounds__(Ring<LOGN>::T, FUSED || PARTS ? 1 : 4) void k_sr_modup(SrUp a, const DevPrime* __restrict__ pr,
                                                            const double* __restrict__ twf,
                                                            const double* __restrict__ twi,
                                                            const double* __restrict__ hat,
                                                            const double* __restrict__ scale) {
  using G = Ring<LOGN>;
  __shared__ double sm[G::LDS];
  const int i = blockIdx.x / a.np, t = blockIdx.x % a.np, b = blockIdx.y, tid = threadIdx.x;
  const int lo = i * ALPHA, nl = a.L - lo < ALPHA ? a.L - lo : ALPHA;
  if (t >= lo && t < lo + nl) return;
  const double q = pr[t].q, qinv = pr[t].qinv;
  double* ext = a.ext + ((size_t)b * a.dnum + i) * a.np * G::N;
  constexpr bool PRE = FUSED || PARTS;
  Fwd<LOGN, PARTS, PRE> f;
  double x[16];
  if constexpr (FUSED) {
    const double qi = pr[i].q, qiv = pr[i].qinv, sc = scale[i], scp = sc * qiv;
    const double* __restrict__ wi = twi + (size_t)i * G::N;
    load_limb<LOGN>(x, a.src + (b / a.inner) * a.outer_st + (b % a.inner) * a.inner_st + (size_t)i * G::N);
    Twiddles<LOGN, PRE> ti;
    load_twiddles<LOGN, PRE>(ti, wi);
    f.load(twf + (size_t)t * G::N, blockIdx.z);
    inv_limb<LOGN, PRE>(x, ti, wi, qi, qiv, sm);
    // one limb: the conversion factor is 1
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = reduce(canon_full(mulc(x[m], sc, scp, qi), qi, qiv), q, qinv);
  } else {
    f.load(twf + (size_t)t * G::N, blockIdx.z);
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = 0.0;
#pragma unroll
    for (int j = 0; j < ALPHA; ++j) {
      if (j >= nl) break;
      const double h = hat[((size_t)i * ALPHA + j) * a.np + t], hp = h * qinv;
      const double* __restrict__ y = ext + (size_t)(lo + j) * G::N;
#pragma unroll
      for (int m = 0; m < 16; ++m) x[m] += mulc(y[tid + G::T * m], h, hp, q);
    }
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = reduce(x[m], q, qinv);
  }
  f.run(x, q, qinv, sm);
  double* o = ext + (size_t)t * G::N + f.base();
#pragma unroll
  for (int m = 0; m < f.WORDS; ++m) o[tid + G::T * m] = canon_full(sm[pad(tid + G::T * m)], q, qinv);
}

// ---------------------------------------------------------------------------
// key switch and ModDown
// ---------------------------------------------------------------------------
struct SrArgs {
  fa::SrItem it[FA_MAXSR];
  int L, np, alpha, dnum;
};

// u[m] = sum_i sigma(ext_i) key_i[h] on prime t at word base + tid + T m, within
// 0.75 dnum q <= 6q.  own: the digit read from c1 (-1: none).  PRE: the next
// digit's words are loaded before the current one's products, as with one
// workgroup on a CU nothing else hides their latency.
template <int LOGN, int W, bool PRE>
__device__ __forceinline__ void key_sum(double (&u)[W], const fa::SrItem& it, int h, int t, int own, int base, int np,
                                        int dnum, double q, double qinv) {
  using G = Ring<LOGN>;
  const int k0 = base + (int)threadIdx.x;
  auto src = [&](int i) { return i == own ? it.c1 + (size_t)t * G::N : it.ext + ((size_t)i * np + t) * G::N; };
  auto key = [&](int i) { return it.key + (((size_t)i * 2 + h) * np + t) * G::N + k0; };
#pragma unroll
  for (int m = 0; m < W; ++m) u[m] = 0.0;
  if constexpr (PRE) {
    uint32_t kk[W];
#pragma unroll
    for (int m = 0; m < W; ++m) kk[m] = perm((uint32_t)(k0 + G::T * m), it.gal, LOGN);
    double x[W], k[W];
    auto load = [&](int i) {
      const double* __restrict__ s = src(i);
      const double* __restrict__ y = key(i);
#pragma unroll
      for (int m = 0; m < W; ++m) {
        x[m] = s[kk[m]];
        k[m] = y[G::T * m];
      }
    };
    load(0);
#pragma unroll 1
    for (int i = 0; i < dnum; ++i) {
      double xc[W], kc[W];
#pragma unroll
      for (int m = 0; m < W; ++m) {
        xc[m] = x[m];
        kc[m] = k[m];
      }
      if (i + 1 < dnum) load(i + 1);
#pragma unroll
      for (int m = 0; m < W; ++m) u[m] += mul(xc[m], kc[m], q, qinv);
    }
  } else {
#pragma unroll 1
    for (int i = 0; i < dnum; ++i) {
      const double* __restrict__ s = src(i);
      const double* __restrict__ y = key(i);
#pragma unroll
      for (int m = 0; m < W; ++m)
        u[m] += mul(s[perm((uint32_t)(k0 + G::T * m), it.gal, LOGN)], y[G::T * m], q, qinv);
    }
  }
}

// Both polynomials' key-switch sums on the special primes, one thread a word,
// at it.y + h * it.yst + k * N: where the inverse transform is repeated by every
// workgroup that needs it, its input is formed once, by enough workgroups to
// fill the chip (one CU reads the keys at little more than 100 GB/s).
template <int DNUM>
__global__ __launch_bounds__(256) void k_sr_special(SrArgs a, const DevPrime* __restrict__ pr, int logn) {
  const int n = 1 << logn;
  const uint32_t k = blockIdx.x * 256 + threadIdx.x;
  const int t = a.L + blockIdx.y;
  const fa::SrItem& it = a.it[blockIdx.z];
  const double q = pr[t].q, qinv = pr[t].qinv;
  const uint32_t kk = perm(k, it.gal, logn);
  double x[DNUM], kb[DNUM], ka[DNUM];
#pragma unroll
  for (int i = 0; i < DNUM; ++i) {
    x[i] = it.ext[((size_t)i * a.np + t) * n + kk];
    kb[i] = it.key[(((size_t)i * 2 + 0) * a.np + t) * n + k];
    ka[i] = it.key[(((size_t)i * 2 + 1) * a.np + t) * n + k];
  }
  double s0 = 0.0, s1 = 0.0;
#pragma unroll
  for (int i = 0; i < DNUM; ++i) {
    s0 += mul(x[i], kb[i], q, qinv);
    s1 += mul(x[i], ka[i], q, qinv);
  }
  double* y = it.y + (size_t)blockIdx.y * n + k;
  y[0] = canon_full(s0, q, qinv);
  y[it.yst] = canon_full(s1, q, qinv);
}

// Special primes: the coefficients of the key-switch sum, scaled for the
// conversion, at it.y + h * it.yst + k * N.  SUM false: the sum is read from it.u
// ([2][np][N]) instead of formed here (it.y may then be its special limbs).
template <int LOGN, bool SUM, bool PRE>
__global__ __launch_bounds__(Ring<LOGN>::T, PRE ? 1 : 4) void k_sr_ksinv(SrArgs a, const DevPrime* __restrict__ pr,
                                                            const double* __restrict__ twi,
                                                            const double* __restrict__ scale) {
  using G = Ring<LOGN>;
  __shared__ double sm[G::LDS];
  const int K = a.np - a.L, h = blockIdx.x / K, k = blockIdx.x % K, t = a.L + k, tid = threadIdx.x;
  const fa::SrItem& it = a.it[blockIdx.y];
  const double q = pr[t].q, qinv = pr[t].qinv, sc = scale[k], scp = sc * qinv;
  const double* __restrict__ w = twi + (size_t)t * G::N;
  Twiddles<LOGN, PRE> tt;
  load_twiddles<LOGN, PRE>(tt, w);
  double x[16];
  if constexpr (SUM) {
    key_sum<LOGN, 16, PRE>(x, it, h, t, -1, 0, a.np, a.dnum, q, qinv);
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = reduce(x[m], q, qinv);
  } else {
    load_limb<LOGN>(x, it.u + ((size_t)h * a.np + t) * G::N);
  }
  inv_limb<LOGN, PRE>(x, tt, w, q, qinv, sm);
  double* y = it.y + h * it.yst + (size_t)k * G::N;
#pragma unroll
  for (int m = 0; m < 16; ++m) y[tid + G::T * m] = canon_full(mulc(x[m], sc, scp, q), q, qinv);
}

// Ciphertext primes: conversion of the special primes' coefficients to prime t,
// its forward transform, then
//   out_h = (u_h - conv_h^) P^-1 + [h = 0] sigma(c0) + add_h
// with u_h formed here (SUM) or read from it.u.  FUSED (one special prime, SUM):
// it.y holds the special prime's sums, whose inverse transform runs here too.
template <int LOGN, int KP, bool SUM, bool FUSED, bool PARTS>
__global__ __launch_bounds__(Ring<LOGN>::T, FUSED || PARTS ? 1 : 4) void k_sr_finish(SrArgs a, const DevPrime* __restrict__ pr,
                                                             const double* __restrict__ twf,
                                                             const double* __restrict__ twi,
                                                             const double* __restrict__ hat,
                                                             const double* __restrict__ scale) {
  using G = Ring<LOGN>;
  __shared__ double sm[G::LDS];
  const int h = blockIdx.x / a.L, t = blockIdx.x % a.L, tid = threadIdx.x;
  const fa::SrItem& it = a.it[blockIdx.y];
  const double q = pr[t].q, qinv = pr[t].qinv;
  constexpr bool PRE = FUSED || PARTS;
  Fwd<LOGN, PARTS, PRE> f;
  double x[16];
  if constexpr (FUSED) {
    const double qk = pr[a.L].q, qkv = pr[a.L].qinv, sc = scale[0], scp = sc * qkv;
    const double* __restrict__ wi = twi + (size_t)a.L * G::N;
    load_limb<LOGN>(x, it.y + h * it.yst);
    Twiddles<LOGN, PRE> ti;
    load_twiddles<LOGN, PRE>(ti, wi);
    f.load(twf + (size_t)t * G::N, blockIdx.z);
    inv_limb<LOGN, PRE>(x, ti, wi, qk, qkv, sm);
    // one special prime: the conversion factor is 1
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = reduce(canon_full(mulc(x[m], sc, scp, qk), qk, qkv), q, qinv);
  } else {
    f.load(twf + (size_t)t * G::N, blockIdx.z);
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = 0.0;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const double c = hat[(size_t)j * a.L + t], cp = c * qinv;
      const double* __restrict__ y = it.y + h * it.yst + (size_t)j * G::N;
#pragma unroll
      for (int m = 0; m < 16; ++m) x[m] += mulc(y[tid + G::T * m], c, cp, q);
    }
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = reduce(x[m], q, qinv);
  }
  f.run(x, q, qinv, sm);
  constexpr int W = decltype(f)::WORDS;
  const int k0 = f.base() + tid;
  const size_t o = (size_t)t * G::N, oh = ((size_t)h * a.L + t) * G::N;
  double u[W];
  if constexpr (SUM) {
    key_sum<LOGN, W, PRE>(u, it, h, t, t / a.alpha, f.base(), a.np, a.dnum, q, qinv);
#pragma unroll
    for (int m = 0; m < W; ++m) u[m] = reduce(u[m], q, qinv);
  } else {
#pragma unroll
    for (int m = 0; m < W; ++m) u[m] = it.u[((size_t)h * a.np + t) * G::N + k0 + G::T * m];
  }
  const double pv = pr[t].pinv, pvp = pv * qinv;
  const bool c0 = h == 0 && it.c0;
  const double* __restrict__ add = it.add[h];
#pragma unroll
  for (int m = 0; m < W; ++m) {
    const int k = k0 + G::T * m;
    // SUM: |u| <= q/2 and the transform within 7.5 q; else u canonical, so the
    // transform's word is reduced first
    const double z = sm[pad(tid + G::T * m)];
    double r = SUM ? mulc(u[m] - z, pv, pvp, q) : mulc(u[m] - reduce(z, q, qinv), pv, pvp, q);
    if (c0) r += it.c0[o + perm((uint32_t)k, it.gal, LOGN)];
    if (add) r += add[o + k];
    it.out[oh + k] = canon_full(r, q, qinv);
  }
}

// Key-switch sums of the giant steps on every prime, u[blk] = sum_g ( sum_i
// sigma_g(ext[blk][g]_i) key_g[i] + P sigma_g(acc_g.c0) ), one thread a word.
struct SrGiant {
  const double* ext;  // [nb][ngs][dnum][np][N]
  const double* acc;  // acc_g of block blk at acc + blk * astride + g * 2 L N
  double* u;          // [nb][2][np][N]
  size_t astride;
  int g0, ng, ngs, L, np, alpha;  // giants g0 + 1 .. g0 + ng of ngs; added to u when g0 > 0
  uint32_t gal[FA_MAXSRG];
  const double* key[FA_MAXSRG];
};
static_assert(sizeof(SrGiant) <= 4000 && sizeof(SrArgs) <= 4000, "kernel arguments");

template <int DNUM>
__global__ __launch_bounds__(256) void k_sr_giant(SrGiant a, const DevPrime* __restrict__ pr, int logn) {
  const int n = 1 << logn;
  const uint32_t k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y, blk = blockIdx.z;
  const double q = pr[t].q, qinv = pr[t].qinv, pm = pr[t].pmod;
  const int own = t < a.L ? t / a.alpha : -1;
  double s0 = 0.0, s1 = 0.0;
#pragma unroll 1
  for (int g = 0; g < a.ng; ++g) {
    const uint32_t kk = perm(k, a.gal[g], logn);
    const double* __restrict__ accg = a.acc + (size_t)blk * a.astride + (size_t)(a.g0 + g + 1) * 2 * a.L * n;
    const double* __restrict__ ext = a.ext + ((size_t)blk * a.ngs + a.g0 + g) * DNUM * a.np * n;
    const double* __restrict__ key = a.key[g];
    double x[DNUM], kb[DNUM], ka[DNUM];
#pragma unroll
    for (int i = 0; i < DNUM; ++i) {
      x[i] = i == own ? accg[((size_t)a.L + t) * n + kk] : ext[((size_t)i * a.np + t) * n + kk];
      kb[i] = key[(((size_t)i * 2 + 0) * a.np + t) * n + k];
      ka[i] = key[(((size_t)i * 2 + 1) * a.np + t) * n + k];
    }
    const double c0 = t < a.L ? accg[(size_t)t * n + kk] : 0.0;
#pragma unroll
    for (int i = 0; i < DNUM; ++i) {
      s0 += mul(x[i], kb[i], q, qinv);
      s1 += mul(x[i], ka[i], q, qinv);
    }
    // at most 0.5 + (8 + 1) 0.75 < 8
    s0 = reduce(s0 + mul(c0, pm, q, qinv), q, qinv);
    s1 = reduce(s1, q, qinv);
  }
  double* u0 = a.u + ((size_t)blk * 2 * a.np + t) * n + k;
  double* u1 = u0 + (size_t)a.np * n;
  if (a.g0) {
    s0 += *u0;
    s1 += *u1;
  }
  *u0 = canon_full(s0, q, qinv);
  *u1 = canon_full(s1, q, qinv);
}

// Rescale by the last prime: the centred lift of its coefficients to prime t,
// the forward transform, out = (ct - lift^) q_last^-1.
template <int LOGN, bool PRE>
__global__ __launch_bounds__(Ring<LOGN>::T, PRE ? 1 : 4) void k_sr_rescale(const double* __restrict__ ct,
                                                              const double* __restrict__ last,
                                                              double* __restrict__ out, fa::SrRes res,
                                                              const DevPrime* __restrict__ pr,
                                                              const double* __restrict__ twf, int L) {
  using G = Ring<LOGN>;
  __shared__ double sm[G::LDS];
  const int t = blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
  const double q = pr[t].q, qinv = pr[t].qinv, ql = pr[L - 1].q;
  const double* __restrict__ w = twf + (size_t)t * G::N;
  Twiddles<LOGN, PRE> tt;
  load_twiddles<LOGN, PRE>(tt, w);
  double x[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    double v = last[(size_t)h * G::N + tid + G::T * m];
    if (v > 0.5 * (ql - 1.0)) v -= ql;
    x[m] = reduce(v, q, qinv);
  }
  fwd_limb<LOGN, PRE>(x, tt, w, q, qinv, sm);
  const double c = res.c[t], cp = c * qinv;
  const double* __restrict__ in = ct + ((size_t)h * L + t) * G::N;
  double* __restrict__ o = out + ((size_t)h * (L - 1) + t) * G::N;
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int k = tid + G::T * m;
    o[k] = canon_full(mulc(in[k] - reduce(sm[pad(k)], q, qinv), c, cp, q), q, qinv);
  }
}

// Full twiddle tables psi^brev(k), k < N, of every prime from the two-pass
// tables: w(s, j) is the product of a row factor and a table entry for stages
// past SA = logn - 8, and the first table below.
__global__ __launch_bounds__(256) void k_sr_tables(double* __restrict__ tw, const double* __restrict__ twa,
                                                   const double* __restrict__ twt, const double* __restrict__ twr,
                                                   const DevPrime* __restrict__ pr, int logn) {
  const int n = 1 << logn, SA = logn - 8;
  const int k = blockIdx.x * 256 + threadIdx.x, t = blockIdx.y;
  const double q = pr[t].q, qinv = pr[t].qinv;
  double w;
  if (k < 256) {
    w = twa[(size_t)t * 256 + k];
  } else {
    const int s = 31 - __clz(k), s1 = s - SA, j = k - (1 << s);  // stage and twiddle index within it
    const int r = j >> s1, i1 = j & ((1 << s1) - 1);
    w = canon_full(mul(twt[(size_t)t * 256 + (1 << s1) + i1], twr[((size_t)t * (n >> 8) + r) * 8 + s1], q, qinv), q,
                   qinv);
  }
  tw[(size_t)t * n + k] = w;
}

}  // namespace

// ===========================================================================
// launchers
// ===========================================================================
namespace fa {

#define FA_SR_SWITCH(fn, ...)         \
  switch (c->logn) {                   \
    case 10: fn<10>(__VA_ARGS__); break; \
    case 11: fn<11>(__VA_ARGS__); break; \
    case 12: fn<12>(__VA_ARGS__); break; \
    case 13: fn<13>(__VA_ARGS__); break; \
    default: break;                    \
  }

void sr_tables(const fa_ctx* c, hipStream_t s) {
  const dim3 g(c->n / 256, c->np);
  hipLaunchKernelGGL(k_sr_tables, g, dim3(256), 0, s, c->d_tws_fwd, c->d_twa_fwd, c->d_twt_fwd, c->d_twr_fwd, c->d_pr,
                     c->logn);
  hipLaunchKernelGGL(k_sr_tables, g, dim3(256), 0, s, c->d_tws_inv, c->d_twa_inv, c->d_twt_inv, c->d_twr_inv, c->d_pr,
                     c->logn);
}

template <int LOGN>
static void launch_list(const fa_ctx* c, const LimbList& l, bool fwd, hipStream_t s) {
  if (fwd)
    hipLaunchKernelGGL(k_sr_fwd_list<LOGN>, dim3(l.n), dim3(Ring<LOGN>::T), 0, s, l, c->d_pr, c->d_tws_fwd);
  else
    hipLaunchKernelGGL(k_sr_inv_list<LOGN>, dim3(l.n), dim3(Ring<LOGN>::T), 0, s, l, c->d_pr, c->d_tws_inv);
}
void sr_ntt(const fa_ctx* c, const LimbList& l, bool fwd, hipStream_t s) {
  if (l.n) FA_SR_SWITCH(launch_list, c, l, fwd, s)
}

// Workgroups up to which a launch repeats work to spread it: the one-limb
// inverse transforms (instead of a launch of their own) and, by parts, the first
// two forward stages.  Up to one workgroup per CU the repeats cost no time; with
// two per CU (their LDS fits twice) quartered transforms still gain.
static constexpr int kSrFused = 256, kSrParts = 512;

template <int LOGN, int ALPHA>
static void launch_modup(const fa_ctx* c, const SrUp& a, int count, hipStream_t s) {
  const int wgs = c->dnum * (c->np - ALPHA) * count;
  const bool parts = kParts * wgs <= kSrParts;
  const dim3 g(c->dnum * c->np, count, parts ? kParts : 1), b(Ring<LOGN>::T);
  auto run = [&](auto fused, auto pt) {
    hipLaunchKernelGGL((k_sr_modup<LOGN, ALPHA, decltype(fused)::value, decltype(pt)::value>), g, b, 0, s, a, c->d_pr,
                       c->d_tws_fwd, c->d_tws_inv, c->d_mu_hat, c->d_mu_scale);
  };
  using Y = std::true_type;
  using Z = std::false_type;
  if constexpr (ALPHA == 1) {
    if (wgs <= kSrFused) return parts ? run(Y{}, Y{}) : run(Y{}, Z{});
  }
  if (c->L * count <= kSrFused)
    hipLaunchKernelGGL((k_sr_inv<LOGN, true>), dim3(c->L, count), b, 0, s, a, c->d_pr, c->d_tws_inv, c->d_mu_scale);
  else
    hipLaunchKernelGGL((k_sr_inv<LOGN, false>), dim3(c->L, count), b, 0, s, a, c->d_pr, c->d_tws_inv, c->d_mu_scale);
  parts ? run(Z{}, Y{}) : run(Z{}, Z{});
}
template <int LOGN>
static void launch_modup_alpha(const fa_ctx* c, const SrUp& a, int count, hipStream_t s) {
  switch (c->alpha) {
    case 1: launch_modup<LOGN, 1>(c, a, count, s); break;
    case 2: launch_modup<LOGN, 2>(c, a, count, s); break;
    case 3: launch_modup<LOGN, 3>(c, a, count, s); break;
    case 4: launch_modup<LOGN, 4>(c, a, count, s); break;
    default: break;
  }
}

void sr_modup(const fa_ctx* c, const double* src, size_t outer_st, int outer, size_t inner_st, int inner, double* ext,
              hipStream_t s) {
  const size_t ext_w = (size_t)c->dnum * c->np * c->n;
  // grid.y is at most 65535: whole outer items per launch
  const int per = std::max(1, 65535 / inner);
  for (int o0 = 0; o0 < outer; o0 += per) {
    const int m = std::min(per, outer - o0);
    const SrUp a{src + (size_t)o0 * outer_st, ext + (size_t)o0 * inner * ext_w, outer_st, inner_st, inner, c->L,
                 c->np, c->alpha, c->dnum};
    FA_SR_SWITCH(launch_modup_alpha, c, a, m * inner, s)
  }
}

template <int DNUM>
static void launch_special(const fa_ctx* c, const SrArgs& a, int m, hipStream_t s) {
  hipLaunchKernelGGL(k_sr_special<DNUM>, dim3(c->n / 256, c->K, m), dim3(256), 0, s, a, c->d_pr, c->logn);
}
#define FA_DNUM_SWITCH(fn, ...)      \
  switch (c->dnum) {                 \
    case 1: fn<1>(__VA_ARGS__); break; \
    case 2: fn<2>(__VA_ARGS__); break; \
    case 3: fn<3>(__VA_ARGS__); break; \
    case 4: fn<4>(__VA_ARGS__); break; \
    case 5: fn<5>(__VA_ARGS__); break; \
    case 6: fn<6>(__VA_ARGS__); break; \
    case 7: fn<7>(__VA_ARGS__); break; \
    case 8: fn<8>(__VA_ARGS__); break; \
    default: break;                  \
  }

template <int LOGN, int KP>
static void launch_finish(const fa_ctx* c, const SrArgs& a, int m, bool sum, hipStream_t s) {
  const int wgs = 2 * c->L * m;
  const bool parts = kParts * wgs <= kSrParts;
  const dim3 g(2 * c->L, m, parts ? kParts : 1), b(Ring<LOGN>::T), gi(2 * c->K, m);
  using Y = std::true_type;
  using Z = std::false_type;
  auto run = [&](auto sm, auto fused, auto pt) {
    hipLaunchKernelGGL((k_sr_finish<LOGN, KP, decltype(sm)::value, decltype(fused)::value, decltype(pt)::value>), g, b,
                       0, s, a, c->d_pr, c->d_tws_fwd, c->d_tws_inv, c->d_md_hat, c->d_md_scale);
  };
  if constexpr (KP == 1) {
    if (sum && wgs <= kSrFused) {
      FA_DNUM_SWITCH(launch_special, c, a, m, s)
      return parts ? run(Y{}, Y{}, Y{}) : run(Y{}, Y{}, Z{});
    }
  }
  auto inv = [&](auto sm, auto pre) {
    hipLaunchKernelGGL((k_sr_ksinv<LOGN, decltype(sm)::value, decltype(pre)::value>), gi, b, 0, s, a, c->d_pr,
                       c->d_tws_inv, c->d_md_scale);
  };
  const bool pre = 2 * c->K * m <= kSrFused;
  if (sum) {
    pre ? inv(Y{}, Y{}) : inv(Y{}, Z{});
    parts ? run(Y{}, Z{}, Y{}) : run(Y{}, Z{}, Z{});
  } else {
    pre ? inv(Z{}, Y{}) : inv(Z{}, Z{});
    parts ? run(Z{}, Z{}, Y{}) : run(Z{}, Z{}, Z{});
  }
}
template <int LOGN>
static void launch_finish_k(const fa_ctx* c, const SrArgs& a, int m, bool sum, hipStream_t s) {
  switch (c->K) {
    case 1: launch_finish<LOGN, 1>(c, a, m, sum, s); break;
    case 2: launch_finish<LOGN, 2>(c, a, m, sum, s); break;
    case 3: launch_finish<LOGN, 3>(c, a, m, sum, s); break;
    case 4: launch_finish<LOGN, 4>(c, a, m, sum, s); break;
    default: break;
  }
}

void sr_finish(const fa_ctx* c, const SrItem* items, int count, bool sum, hipStream_t s) {
  for (int j0 = 0; j0 < count; j0 += FA_MAXSR) {
    const int m = std::min(FA_MAXSR, count - j0);
    SrArgs a;
    for (int j = 0; j < m; ++j) a.it[j] = items[j0 + j];
    a.L = c->L;
    a.np = c->np;
    a.alpha = c->alpha;
    a.dnum = c->dnum;
    FA_SR_SWITCH(launch_finish_k, c, a, m, sum, s)
  }
}

template <int DNUM>
static void launch_giant(const fa_ctx* c, const SrGiant& a, int nb, hipStream_t s) {
  hipLaunchKernelGGL(k_sr_giant<DNUM>, dim3(c->n / 256, c->np, nb), dim3(256), 0, s, a, c->d_pr, c->logn);
}
void sr_giant(const fa_ctx* c, const double* ext, const double* acc, size_t astride, const double* const* keys,
              const uint32_t* gals, int nb, int ng, double* u, hipStream_t s) {
  for (int g0 = 0; g0 < ng; g0 += FA_MAXSRG) {
    SrGiant a{ext, acc, u, astride, g0, std::min(FA_MAXSRG, ng - g0), ng, c->L, c->np, c->alpha, {}, {}};
    for (int g = 0; g < a.ng; ++g) {
      a.gal[g] = gals[g0 + g];
      a.key[g] = keys[g0 + g];
    }
    FA_DNUM_SWITCH(launch_giant, c, a, nb, s)
  }
}

template <int LOGN>
static void launch_rescale(const fa_ctx* c, const double* ct, const double* last, int n_polys, double* out,
                           const SrRes& r, hipStream_t s) {
  const dim3 g(c->L - 1, n_polys), b(Ring<LOGN>::T);
  if ((c->L - 1) * n_polys <= kSrFused)
    hipLaunchKernelGGL((k_sr_rescale<LOGN, true>), g, b, 0, s, ct, last, out, r, c->d_pr, c->d_tws_fwd, c->L);
  else
    hipLaunchKernelGGL((k_sr_rescale<LOGN, false>), g, b, 0, s, ct, last, out, r, c->d_pr, c->d_tws_fwd, c->L);
}
void sr_rescale(const fa_ctx* c, const double* ct, const double* last, int n_polys, double* out, const SrRes& r,
                hipStream_t s) {
  FA_SR_SWITCH(launch_rescale, c, ct, last, n_polys, out, r, s)
}

}  // namespace fa
