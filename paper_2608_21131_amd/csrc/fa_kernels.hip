// HIP kernels of libfa for gfx950 (CDNA4, wave64).
//
// Residue arithmetic in float64.  Every prime q is in (2^49, 2^50); residues
// and lazily reduced values are integers of magnitude < 2^53 held exactly in
// doubles.  A modular product uses the FMA to split a*b exactly into
// h = fl(a*b) and l = a*b - h, estimates the quotient t = rint(a*b/q) from a
// precomputed 1/q (or w/q), and forms a*b - t*q = fma(-t, q, h) + l, which is
// exact because the true value is an integer below 2^53.  fp64 FMA issues at
// full rate on CDNA while 32-bit integer multiplies issue at quarter rate,
// which is why the residues are doubles and not u64.
//
// Bounds used below (u = 2^-53, all q in (2^49, 2^50)):
//   mulc(a, w, w/q):  for |a| <= c*q the quotient estimate is off by at most
//     0.375c, so |result| <= (0.5 + 0.375c) q; exact for |a| <= 8q.
//   mul(a, b):        |a|, |b| <= q  ->  |result| <= 0.75 q.
//   mul(a, w) with |a| <= c*q and |w| <= q bounds the same way as mulc: its
//     quotient estimate carries the same three roundings.
//   reduce(x):        |x| < 2^53    ->  |result| <= q/2 (+ rounding slack).
// Forward NTT values stay within 7.8 q (see ct_bfly and col_reduces), inverse
// NTT values within 4 q (see gs_bfly); every transform output that leaves a
// kernel is either canonicalised or feeds a mulc / mul whose operand stays
// within 8 q.
// Sums of up to eight products of canonical words stay within 6 q; the giant
// steps' sums, over words of a row pass, are reduced after four (add_digit).

#include <hip/hip_runtime.h>

#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "fa_arith.h"
#include "fa_internal.h"

namespace {

// Cooley-Tukey butterfly (forward): (x, y) -> (x + w y, x - w y).  With R
// false x is not reduced first.  With c the bound (in units of q) of the stage's
// inputs, a reduced stage leaves 1 + 0.375c and a lazy one 1.375c + 0.5.  The row
// passes alternate lazy and reduced stages, lazy first: from the 5.3 that the
// fused column passes may leave (col_reduces) they reach 7.8 once and fall to
// 3.9, 5.9, 3.2, ...; the plain column passes alternate too and leave at most
// 3.9.  Always inside the 8q of the product's exactness and below 2^53.
template <bool R = true>
__device__ __forceinline__ void ct_bfly(double& x, double& y, double w, double q, double qinv) {
  const double u = R ? reduce(x, q, qinv) : x;
  const double t = mul(y, w, q, qinv);
  x = u + t;
  y = u - t;
}
// Gentleman-Sande butterfly (inverse): (x, y) -> (x + y, (x - y) w^-1).  Inputs
// within c give a sum within 2c (reduced to 1/2 unless R is false) and a product
// within 0.5 + 0.75c.  From canonical inputs the row pass leaves its first two
// stages' sums lazy (2, then 4: products of at most 8q are exact) and reduces
// from there on: 3.5, 3.13, 2.85, ... towards 2.
template <bool R = true>
__device__ __forceinline__ void gs_bfly(double& x, double& y, double winv, double q, double qinv) {
  const double u = x + y;
  const double v = x - y;
  x = R ? reduce(u, q, qinv) : u;
  y = mul(v, winv, q, qinv);
}

// ---------------------------------------------------------------------------
// Negacyclic NTT, N = 2^logn = 2^SA * 256, natural order in, bit-reversed out.
// Stage s pairs elements j and j + N/2^(s+1) with twiddle
//   w(s, j) = psi^brev(2^s + (j >> (logn - s)))       (brev over logn bits).
// Pass A runs stages 0..SA-1 on columns (j mod 256 fixed): its twiddles are
// the first 2^SA table entries.  Pass B runs stages SA..SA+7 on contiguous
// rows of 256; for row r and stage SA + s' the twiddle factors as
//   w = f[r][s'] * T[2^s' + i'],  f[r][s'] = psi^((2 brev_SA(r) + 1) 2^(7-s')),
//   T[2^s' + i'] = psi^(brev_s'(i') N / 2^s'),
// so pass B reads 8 row factors and a 256-entry table instead of N entries.
// Each pass keeps a unit of elements in registers for half its stages,
// exchanges through LDS, then finishes.
// ---------------------------------------------------------------------------
template <int SA>
struct PassA {
  static constexpr int H = 1 << SA;
  static constexpr int S1 = (SA + 1) / 2;
  static constexpr int S2 = SA - S1;
  static constexpr int E1 = 1 << S1;
  static constexpr int E2 = 1 << S2;
  static constexpr int COLS = (4096 >> SA) < 256 ? (4096 >> SA) : 256;
  static constexpr int TILE = COLS * H;
};

// loaders for the first pass of the forward transform
struct PlainLd {
  const double* src;
  __device__ double operator()(size_t i) const { return src[i]; }
};
// v mod q within q/2 + 2^32 for any 64-bit v: the high half times 2^32 is exact in
// a double and so is its reduction (the quotient is below 2^14).  A 64-bit integer
// division here takes longer than the pass's eight stages.
__device__ __forceinline__ double int_residue(int64_t v, double q, double qinv) {
  return reduce((double)(int32_t)(v >> 32) * 0x1p32, q, qinv) + (double)(uint32_t)v;
}
struct IntLd {
  const int64_t* src;
  double q, qinv;
  __device__ double operator()(size_t i) const { return int_residue(src[i], q, qinv); }
};
template <int SA, class Ld>
__device__ __forceinline__ void fwd_a_body(const Ld& ld, double* a, const double* __restrict__ w, double q,
                                           double qinv, int col0, double* sm) {
  using P = PassA<SA>;
  for (int u = threadIdx.x; u < P::TILE / P::E1; u += 256) {
    const int c = u % P::COLS, hl = u / P::COLS;
    double x[P::E1];
#pragma unroll
    for (int m = 0; m < P::E1; ++m) x[m] = ld(((size_t)(hl + (m << P::S2)) << 8) + col0 + c);
#pragma unroll
    for (int s = 0; s < P::S1; ++s) {
      const int half = P::E1 >> (s + 1);
#pragma unroll
      for (int m = 0; m < P::E1; ++m) {
        if (m & half) continue;
        if (s & 1) ct_bfly<true>(x[m], x[m + half], w[(1 << s) + (m >> (P::S1 - s))], q, qinv);
        else ct_bfly<false>(x[m], x[m + half], w[(1 << s) + (m >> (P::S1 - s))], q, qinv);
      }
    }
#pragma unroll
    for (int m = 0; m < P::E1; ++m) sm[(hl + (m << P::S2)) * P::COLS + c] = x[m];
  }
  __syncthreads();
  for (int u = threadIdx.x; u < P::TILE / P::E2; u += 256) {
    const int c = u % P::COLS, hh = u / P::COLS;
    double x[P::E2];
#pragma unroll
    for (int m = 0; m < P::E2; ++m) x[m] = sm[((hh << P::S2) + m) * P::COLS + c];
#pragma unroll
    for (int s2 = 0; s2 < P::S2; ++s2) {
      const int s = P::S1 + s2, half = P::E2 >> (s2 + 1);
#pragma unroll
      for (int m = 0; m < P::E2; ++m) {
        if (m & half) continue;
        if (s & 1) ct_bfly<true>(x[m], x[m + half], w[(1 << s) + (hh << s2) + (m >> (P::S2 - s2))], q, qinv);
        else ct_bfly<false>(x[m], x[m + half], w[(1 << s) + (hh << s2) + (m >> (P::S2 - s2))], q, qinv);
      }
    }
#pragma unroll
    for (int m = 0; m < P::E2; ++m) a[((size_t)((hh << P::S2) + m) << 8) + col0 + c] = x[m];
  }
}

template <int SA>
__global__ __launch_bounds__(256) void k_ntt_fwd_a(LimbList ll, const DevPrime* __restrict__ pr,
                                                   const double* __restrict__ twa) {
  using P = PassA<SA>;
  __shared__ double sm[P::TILE];
  const int pi = ll.prime[blockIdx.y];
  const double q = pr[pi].q, qinv = pr[pi].qinv;
  fwd_a_body<SA>(PlainLd{ll.src[blockIdx.y]}, ll.ptr[blockIdx.y], twa + (size_t)pi * 256, q, qinv,
                 blockIdx.x * P::COLS, sm);
}

// The same pass from integer coefficients, prime t = blockIdx.y of polynomial
// blockIdx.z: the residues never go through memory.
template <int SA>
__global__ __launch_bounds__(256) void k_ntt_fwd_a_int(const int64_t* __restrict__ src, double* __restrict__ dst,
                                                       const DevPrime* __restrict__ pr,
                                                       const double* __restrict__ twa, int L) {
  using P = PassA<SA>;
  __shared__ double sm[P::TILE];
  constexpr size_t n = (size_t)P::H << 8;
  const int t = blockIdx.y;
  const double q = pr[t].q, qinv = pr[t].qinv;
  fwd_a_body<SA>(IntLd{src + blockIdx.z * n, q, qinv}, dst + (blockIdx.z * (size_t)L + t) * n, twa + (size_t)t * 256, q,
                 qinv, blockIdx.x * P::COLS, sm);
}

// ModUp, first pass: ext[i][t] = pass A of Conv_{digit i -> t}(y), for every
// digit i and prime t outside the digit.
struct MuArgs {
  fa::MuItem it[FA_MAXMU];
};

// Fused basis conversion from row-passed sources: a workgroup owns one column
// tile of one source group (a digit of c1 for ModUp, the special primes for
// ModDown).  It finishes the inverse transform of the group's limbs on that
// tile (column pass, then the scaling by N^-1 times the conversion factor,
// leaving canonical residues, exactly as k_ntt_inv_a does) and keeps the
// results in registers; then for every target prime it forms the fast basis
// conversion of the tile (as ConvLd does) and runs the first forward pass on
// it (as fwd_a_body does).  Each source word is read once and the
// coefficients never leave the chip.  With ngrp > 1 the targets are split
// into ngrp contiguous groups, one per workgroup (each group repeats the
// inverse pass): small launches get more workgroups.
//
// Src describes the group: nl source limbs src(j) over primes sprime(j) with
// scales scale(j); ntarget targets, the k-th over prime target(k), with
// conversion factors hat(j, t), written to out(t); CENTRE takes the sources'
// representatives around 0 instead of canonical ones.
//
// 512 threads hold eight words each, so the columns take two or three passes of
// two or three stages with an LDS exchange between them.  With sixteen words on
// 256 threads, one exchange, the kept coefficients took 232-256 registers and
// two waves per SIMD; eight words leave room for four (128 registers, of which
// ModDown at N = 2^15 spills 2 with 3 special primes and 6 with 4).  At N = 2^16
// with 12+3 primes a ModDown launch of 16 polynomials went from 91 to 74 us beside
// the other lane's work (its 126 MB are 30 us at a copy's 4.8 TB/s); the rest of
// the gain is in small launches, see conv_groups.
template <int SA>
struct ColPass {
  static constexpr int H = 1 << SA, COLS = 4096 >> SA, T = 512;
  static constexpr int PASSES = SA > 6 ? 3 : 2;
  static constexpr int stages(int p) { return SA == 8 ? (p < 2 ? 3 : 2) : SA == 7 ? (p < 1 ? 3 : 2) : 3; }
  static constexpr int first(int p) { return p == 0 ? 0 : first(p - 1) + stages(p - 1); }
  // row group of unit v and the row of its element m in pass p
  template <int P>
  static __device__ __forceinline__ int group(int v) {
    return ((int)threadIdx.x + T * v) / COLS;
  }
  template <int P>
  static __device__ __forceinline__ int row(int v, int m) {
    constexpr int R = stages(P), ls = SA - first(P) - R;
    const int g = group<P>(v);
    return ((g >> ls) << (ls + R)) + (g & ((1 << ls) - 1)) + (m << ls);
  }
  // LDS word of a row's column: rows 4 or 8 apart land on the other half of the
  // banks (a half-wave reads two 16-word pieces at COLS = 16)
  static __device__ __forceinline__ int lds(int row) {
    const int a = row * COLS + (int)threadIdx.x % COLS;
    return a ^ (((a >> 2) ^ (a >> 3)) & 16);
  }
  // the first twiddle of stage s1 of pass p for unit v: one per wave where a wave
  // lies inside a block of rows
  template <int P>
  static __device__ __forceinline__ int tw(int v, int s1) {
    constexpr int S = first(P), R = stages(P), ls = SA - S - R;
    if constexpr (S == 0) return 1 << s1;
    const int blk = group<P>(v) >> ls;
    constexpr bool uniform = (COLS << ls) >= 64;
    return (1 << (S + s1)) + ((uniform ? __builtin_amdgcn_readfirstlane(blk) : blk) << s1);
  }
};
// Does forward column stage s reduce its first operand?  From |x| <= q/2 (a
// reduced conversion); the row pass takes inputs within 5.3 q, see ct_bfly.
constexpr bool col_reduces(int s) {
  double c = 0.5;
  for (int i = 0;; ++i) {
    const bool r = 1.375 * c + 0.5 > 5.3;
    if (i == s) return r;
    c = r ? 1.0 + 0.375 * c : 1.375 * c + 0.5;
  }
}
template <int SA, int P>
__device__ __forceinline__ void col_put(const double (&x)[8], double* sm) {
  using C = ColPass<SA>;
  constexpr int E = 1 << C::stages(P);
#pragma unroll
  for (int e = 0; e < 8; ++e) sm[C::lds(C::template row<P>(e / E, e % E))] = x[e];
}
template <int SA, int P>
__device__ __forceinline__ void col_get(double (&x)[8], const double* sm) {
  using C = ColPass<SA>;
  constexpr int E = 1 << C::stages(P);
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = sm[C::lds(C::template row<P>(e / E, e % E))];
}
template <int SA, int P>
__device__ __forceinline__ void col_fwd(double (&x)[8], const double* __restrict__ w, double q, double qinv) {
  using C = ColPass<SA>;
  constexpr int S = C::first(P), R = C::stages(P), E = 1 << R;
#pragma unroll
  for (int s1 = 0; s1 < R; ++s1)
#pragma unroll
    for (int v = 0; v < 8 / E; ++v) {
      const int half = E >> (s1 + 1);
      const double* __restrict__ ws = w + C::template tw<P>(v, s1);
#pragma unroll
      for (int m = 0; m < E; ++m) {
        if (m & half) continue;
        if (col_reduces(S + s1)) ct_bfly<true>(x[v * E + m], x[v * E + m + half], ws[m >> (R - s1)], q, qinv);
        else ct_bfly<false>(x[v * E + m], x[v * E + m + half], ws[m >> (R - s1)], q, qinv);
      }
    }
}
template <int SA, int P>
__device__ __forceinline__ void col_inv(double (&x)[8], const double* __restrict__ w, double q, double qinv) {
  using C = ColPass<SA>;
  constexpr int R = C::stages(P), E = 1 << R;
#pragma unroll
  for (int s1 = R - 1; s1 >= 0; --s1)
#pragma unroll
    for (int v = 0; v < 8 / E; ++v) {
      const int half = E >> (s1 + 1);
      const double* __restrict__ ws = w + C::template tw<P>(v, s1);
#pragma unroll
      for (int m = 0; m < E; ++m) {
        if (m & half) continue;
        gs_bfly(x[v * E + m], x[v * E + m + half], ws[m >> (R - s1)], q, qinv);
      }
    }
}
// all passes; x starts in pass P's layout and ends in the last (first) one's
template <int SA, int P = 0>
__device__ __forceinline__ void col_fwd_all(double (&x)[8], const double* __restrict__ w, double q, double qinv,
                                            double* sm) {
  col_fwd<SA, P>(x, w, q, qinv);
  if constexpr (P + 1 < ColPass<SA>::PASSES) {
    col_put<SA, P>(x, sm);
    __syncthreads();
    col_get<SA, P + 1>(x, sm);
    col_fwd_all<SA, P + 1>(x, w, q, qinv, sm);
  }
}
template <int SA, int P = ColPass<SA>::PASSES - 1>
__device__ __forceinline__ void col_inv_all(double (&x)[8], const double* __restrict__ w, double q, double qinv,
                                            double* sm) {
  col_inv<SA, P>(x, w, q, qinv);
  if constexpr (P > 0) {
    col_put<SA, P>(x, sm);
    __syncthreads();
    col_get<SA, P - 1>(x, sm);
    col_inv_all<SA, P - 1>(x, w, q, qinv, sm);
  }
}

template <int SA, int NS, class Src>
__device__ __forceinline__ void conv_fused_body(const Src& sr, const DevPrime* __restrict__ pr,
                                                const double* __restrict__ twa_f, const double* __restrict__ twa_i,
                                                int grp, int ngrp, double* sm) {
  using C = ColPass<SA>;
  constexpr int PL = C::PASSES - 1, EL = 1 << C::stages(PL);
  const int nl = sr.nl;
  const int col = blockIdx.x * C::COLS + (int)threadIdx.x % C::COLS;
  double y[NS][8];
#pragma unroll
  for (int j = 0; j < NS; ++j)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      y[j][e] = j < nl ? sr.src(j)[((size_t)C::template row<PL>(e / EL, e % EL) << 8) + col] : 0.0;
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    if (j < nl) {
      const int pj = sr.sprime(j);
      const double q = pr[pj].q, qinv = pr[pj].qinv;
      col_inv_all<SA>(y[j], twa_i + (size_t)pj * 256, q, qinv, sm);
      const double sc = sr.scale(j), scp = sc * qinv;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        y[j][e] = canon_full(mulc(y[j][e], sc, scp, q), q, qinv);
        if (Src::CENTRE && y[j][e] > 0.5 * (q - 1.0)) y[j][e] -= q;
      }
      __syncthreads();  // the next limb reuses the LDS tile
    }
  }
  const int per = (sr.ntarget + ngrp - 1) / ngrp;  // targets of this group: k0 <= k < k0 + per
  const int k0 = grp * per;
#pragma unroll 1
  for (int k = k0; k < k0 + per && k < sr.ntarget; ++k) {
    const int t = sr.target(k);
    const double q = pr[t].q, qinv = pr[t].qinv;
    double h[NS], hp[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      h[j] = j < nl ? sr.hat(j, t) : 0.0;
      hp[j] = h[j] * qinv;
    }
    double x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < NS; ++j) acc += mulc(y[j][e], h[j], hp[j], q);
      x[e] = reduce(acc, q, qinv);
    }
    col_fwd_all<SA>(x, twa_f + (size_t)t * 256, q, qinv, sm);
    double* __restrict__ a = sr.out(t) + col;
#pragma unroll
    for (int e = 0; e < 8; ++e) a[(size_t)C::template row<PL>(e / EL, e % EL) << 8] = x[e];
    __syncthreads();  // the next target reuses the LDS tile
  }
}

// ModUp sources: digit i of c1, converted to every prime outside the digit
// (own limbs are read from c1 directly by the key-switch kernels)
struct MuSrc {
  const double* y;     // [L][N], row pass of the inverse done
  double* ext;         // [dnum][np][N]
  const double* hatt;  // [dnum][alpha][np]
  const double* sct;   // [L]
  int i, alpha, lo, nl, n, np, ntarget;
  static constexpr bool CENTRE = false;
  __device__ const double* src(int j) const { return y + (size_t)(lo + j) * n; }
  __device__ int sprime(int j) const { return lo + j; }
  __device__ double scale(int j) const { return sct[lo + j]; }
  __device__ int target(int k) const { return k < lo ? k : k + nl; }
  __device__ double hat(int j, int t) const { return hatt[((size_t)i * alpha + j) * np + t]; }
  __device__ double* out(int t) const { return ext + ((size_t)i * np + t) * n; }
};
// ModDown sources: the K special-prime limbs, converted to the L ciphertext primes
struct MdSrc {
  const double* yP;    // [K][N], row pass of the inverse done
  double* conv;        // [L][N]
  const double* hatt;  // [K][L]
  const double* sct;   // [K]
  int L, nl, n, ntarget;
  static constexpr bool CENTRE = false;
  __device__ const double* src(int j) const { return yP + (size_t)j * n; }
  __device__ int sprime(int j) const { return L + j; }
  __device__ double scale(int j) const { return sct[j]; }
  __device__ int target(int k) const { return k; }
  __device__ double hat(int j, int t) const { return hatt[(size_t)j * L + t]; }
  __device__ double* out(int t) const { return conv + (size_t)t * n; }
};

// Rescale sources: the last ciphertext limb, centred, lifted to the others
struct RsSrc {
  const double* last;  // [N], row pass of the inverse done
  double* lift;        // [L-1][N]
  double ninv;
  int nl, prime, n, ntarget;
  static constexpr bool CENTRE = true;
  __device__ const double* src(int) const { return last; }
  __device__ int sprime(int) const { return prime; }
  __device__ double scale(int) const { return ninv; }
  __device__ int target(int k) const { return k; }
  __device__ double hat(int, int) const { return 1.0; }
  __device__ double* out(int t) const { return lift + (size_t)t * n; }
};

template <int SA, int ALPHA>
__global__ __launch_bounds__(512, 4) void k_modup_fused(MuArgs args, const DevPrime* __restrict__ pr,
                                                     const double* __restrict__ twa_f,
                                                     const double* __restrict__ twa_i,
                                                     const double* __restrict__ hat,
                                                     const double* __restrict__ scale, int logn, int L, int np,
                                                     int ngrp) {
  __shared__ double sm[PassA<SA>::TILE];
  const fa::MuItem& it = args.it[blockIdx.z];
  MuSrc sr;
  sr.y = it.y;
  sr.ext = it.ext;
  sr.hatt = hat;
  sr.sct = scale;
  sr.i = blockIdx.y / ngrp;
  sr.alpha = ALPHA;
  sr.lo = sr.i * ALPHA;
  sr.nl = L - sr.lo < ALPHA ? L - sr.lo : ALPHA;  // a short last digit has fewer limbs
  sr.n = 1 << logn;
  sr.np = np;
  sr.ntarget = np - sr.nl;
  conv_fused_body<SA, ALPHA>(sr, pr, twa_f, twa_i, blockIdx.y % ngrp, ngrp, sm);
}

// ModDown, first pass: conv[t] = pass A of Conv_{P -> q_t}(y_P).
struct MdArgs {
  fa::MdItem it[FA_MAXMD];
};

template <int SA, int KP>
__global__ __launch_bounds__(512, 4) void k_moddown_fused(MdArgs args, const DevPrime* __restrict__ pr,
                                                       const double* __restrict__ twa_f,
                                                       const double* __restrict__ twa_i,
                                                       const double* __restrict__ hat,
                                                       const double* __restrict__ scale, int logn, int L,
                                                       int ngrp) {
  __shared__ double sm[PassA<SA>::TILE];
  const fa::MdItem& it = args.it[blockIdx.z];
  MdSrc sr;
  sr.yP = it.yP;
  sr.conv = it.conv;
  sr.hatt = hat;
  sr.sct = scale;
  sr.L = L;
  sr.nl = KP;
  sr.n = 1 << logn;
  sr.ntarget = L;
  conv_fused_body<SA, KP>(sr, pr, twa_f, twa_i, blockIdx.y, ngrp, sm);
}

// Rescale, first pass: lift[h][t] = pass A of the last limb's centred lift
template <int SA>
__global__ __launch_bounds__(512, 4) void k_rescale_fused(const double* __restrict__ last, double* lift,
                                                          const DevPrime* __restrict__ pr,
                                                          const double* __restrict__ twa_f,
                                                          const double* __restrict__ twa_i, int L, int ngrp) {
  __shared__ double sm[PassA<SA>::TILE];
  constexpr int n = 1 << (SA + 8);
  const size_t h = blockIdx.z;
  conv_fused_body<SA, 1>(RsSrc{last + h * n, lift + h * (L - 1) * n, pr[L - 1].ninv, 1, L - 1, n, L - 1}, pr, twa_f,
                         twa_i, blockIdx.y, ngrp, sm);
}

// inverse pass A (the last pass of the inverse transform): columns; the final
// multiply uses a per-limb constant (N^-1, or N^-1 times a basis-conversion
// factor) and leaves canonical residues.
template <int SA>
__global__ __launch_bounds__(256) void k_ntt_inv_a(LimbList ll, const DevPrime* __restrict__ pr,
                                                   const double* __restrict__ twa) {
  using P = PassA<SA>;
  __shared__ double sm[P::TILE];
  const int pi = ll.prime[blockIdx.y];
  double* __restrict__ a = ll.ptr[blockIdx.y];
  const double q = pr[pi].q, qinv = pr[pi].qinv;
  const double* __restrict__ w = twa + (size_t)pi * 256;
  const int col0 = blockIdx.x * P::COLS;
  for (int u = threadIdx.x; u < P::TILE / P::E2; u += 256) {
    const int c = u % P::COLS, hh = u / P::COLS;
    double x[P::E2];
#pragma unroll
    for (int m = 0; m < P::E2; ++m) x[m] = a[((size_t)((hh << P::S2) + m) << 8) + col0 + c];
#pragma unroll
    for (int s2 = P::S2 - 1; s2 >= 0; --s2) {
      const int s = P::S1 + s2, half = P::E2 >> (s2 + 1);
#pragma unroll
      for (int m = 0; m < P::E2; ++m) {
        if (m & half) continue;
        gs_bfly(x[m], x[m + half], w[(1 << s) + (hh << s2) + (m >> (P::S2 - s2))], q, qinv);
      }
    }
#pragma unroll
    for (int m = 0; m < P::E2; ++m) sm[((hh << P::S2) + m) * P::COLS + c] = x[m];
  }
  __syncthreads();
  const double sc = ll.scale[blockIdx.y], scp = sc * qinv;
  for (int u = threadIdx.x; u < P::TILE / P::E1; u += 256) {
    const int c = u % P::COLS, hl = u / P::COLS;
    double x[P::E1];
#pragma unroll
    for (int m = 0; m < P::E1; ++m) x[m] = sm[(hl + (m << P::S2)) * P::COLS + c];
#pragma unroll
    for (int s = P::S1 - 1; s >= 0; --s) {
      const int half = P::E1 >> (s + 1);
#pragma unroll
      for (int m = 0; m < P::E1; ++m) {
        if (m & half) continue;
        gs_bfly(x[m], x[m + half], w[(1 << s) + (m >> (P::S1 - s))], q, qinv);
      }
    }
#pragma unroll
    for (int m = 0; m < P::E1; ++m)
      a[((size_t)(hl + (m << P::S2)) << 8) + col0 + c] = canon_full(mulc(x[m], sc, scp, q), q, qinv);
  }
}

// Pass B: rows of 256 contiguous elements.  Row stride in LDS is 272 words
// (one pad word per 16) so that both access patterns spread over all banks.
#define ROWW 272
__device__ __forceinline__ int lds_row(int rl, int lo) { return rl * ROWW + lo + (lo >> 4); }

// twiddle of pass B for stage SA+s', row r, index i' (see the header above)
__device__ __forceinline__ double twb(const double* __restrict__ T, double f, int s1, int i1, double q, double qinv) {
  const double t = T[(1 << s1) + i1];
  return mulc(t, f, f * qinv, q);
}

// stores for the last pass of the forward transform, one element at a time
// (global index i, lazily reduced value x); the pass hands them out so that
// consecutive threads touch consecutive words.
struct CanonSt {
  double* a;
  double q, qinv;
  struct Op {};
  __device__ Op load(size_t) const { return {}; }
  __device__ void operator()(size_t i, double x, Op) const { a[i] = canon_full(x, q, qinv); }
};
// ModDown finish: out[k] = base[pi(k)] + (u_Q[k] - conv^[k]) * P^-1
struct FinishSt {
  const double* uQ;
  const double* base;
  double* out;
  uint32_t gal;
  int logn;
  double q, qinv, pv, pvp;
  struct Op {
    double u, b;
  };
  __device__ Op load(size_t i) const {
    return {uQ[i], base ? base[gal == 1u ? (uint32_t)i : perm((uint32_t)i, gal, logn)] : 0.0};
  }
  __device__ void operator()(size_t i, double x, Op o) const {
    out[i] = canon_full(mulc(o.u - x, pv, pvp, q) + o.b, q, qinv);
  }
};

// The eight stages of pass B over `rows` rows row0.. of a; the results are
// left in LDS (lds_row layout) and the block is synchronised on return.
__device__ __forceinline__ void fwd_b_lds(const double* __restrict__ a, int row0, int rows,
                                          const double* __restrict__ T, const double* __restrict__ F, double q,
                                          double qinv, double* sm) {
  for (int u = threadIdx.x; u < rows * 16; u += 256) {
    const int l0 = u & 15, rl = u >> 4, r = row0 + rl;
    double x[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = a[(size_t)r * 256 + l0 + 16 * m];
#pragma unroll
    for (int s1 = 0; s1 < 4; ++s1) {
      const int half = 8 >> s1;
      const double f = F[r * 8 + s1];
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        if (m & half) continue;
        if (s1 & 1) ct_bfly<true>(x[m], x[m + half], twb(T, f, s1, m >> (4 - s1), q, qinv), q, qinv);
        else ct_bfly<false>(x[m], x[m + half], twb(T, f, s1, m >> (4 - s1), q, qinv), q, qinv);
      }
    }
#pragma unroll
    for (int m = 0; m < 16; ++m) sm[lds_row(rl, l0 + 16 * m)] = x[m];
  }
  __syncthreads();
  for (int u = threadIdx.x; u < rows * 16; u += 256) {
    const int lh = u & 15, rl = u >> 4, r = row0 + rl;
    double x[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = sm[lds_row(rl, 16 * lh + m)];
#pragma unroll
    for (int s1 = 4; s1 < 8; ++s1) {
      const int half = 8 >> (s1 - 4);
      const double f = F[r * 8 + s1];
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        if (m & half) continue;
        const double w = twb(T, f, s1, (lh << (s1 - 4)) + (m >> (8 - s1)), q, qinv);
        if (s1 & 1) ct_bfly<true>(x[m], x[m + half], w, q, qinv);
        else ct_bfly<false>(x[m], x[m + half], w, q, qinv);
      }
    }
    // back to LDS: each thread rewrites the words it read
#pragma unroll
    for (int m = 0; m < 16; ++m) sm[lds_row(rl, 16 * lh + m)] = x[m];
  }
  __syncthreads();
}

template <class St>
__device__ __forceinline__ void fwd_b_body(double* a, const St& st, const double* __restrict__ T,
                                           const double* __restrict__ F, double q, double qinv, int logn,
                                           double* sm) {
  // 16 on every ring that comes here (N >= 2^14), but not as a constant: with one,
  // all callers of fwd_b_lds pass at most 16 rows, the compiler drops its loops
  // before it inlines it, and k_giant_ks comes out at 160 registers instead of 206
  // and slower.  Three blocks at N = 2^14, 8+1 primes, d = 64, B = 8: 670 against
  // 429 us; a rerank level 5423 against 4841 us.
  const int rows = (1 << logn >> 8) < 16 ? (1 << logn >> 8) : 16;
  const int row0 = blockIdx.x * rows;
  fwd_b_lds(a, row0, rows, T, F, q, qinv, sm);
  // out with consecutive threads on consecutive words, the finish's operands
  // loaded FIN words at a time: the stores may alias them for all the compiler
  // knows, so word by word every row waited for its own load.  Together with the
  // same in k_moddown_ks_b: a product with its rescale at N = 2^16, 12 primes
  // 147.3 -> 139.4 us, a rerank level at 3 primes 1217 -> 1191 us, a membership
  // scan 6.08 -> 5.97 ms
  constexpr int FIN = 4;  // divides the rows
  const size_t i0 = (size_t)row0 * 256 + threadIdx.x;
  for (int r = 0; r < rows; r += FIN) {
    typename St::Op o[FIN];
#pragma unroll
    for (int j = 0; j < FIN; ++j) o[j] = st.load(i0 + 256 * (r + j));
#pragma unroll
    for (int j = 0; j < FIN; ++j) st(i0 + 256 * (r + j), sm[lds_row(r + j, threadIdx.x)], o[j]);
  }
}

__global__ __launch_bounds__(256) void k_ntt_fwd_b(LimbList ll, const DevPrime* __restrict__ pr,
                                                   const double* __restrict__ twt, const double* __restrict__ twr,
                                                   int logn) {
  __shared__ double sm[16 * ROWW];
  const int pi = ll.prime[blockIdx.y];
  double* a = ll.ptr[blockIdx.y];
  const double q = pr[pi].q, qinv = pr[pi].qinv;
  const int H = 1 << (logn - 8);
  fwd_b_body(a, CanonSt{a, q, qinv}, twt + (size_t)pi * 256, twr + (size_t)pi * H * 8, q, qinv, logn, sm);
}

__global__ __launch_bounds__(256) void k_moddown_b(MdArgs args, const DevPrime* __restrict__ pr,
                                                   const double* __restrict__ twt, const double* __restrict__ twr,
                                                   int logn) {
  __shared__ double sm[16 * ROWW];
  const int t = blockIdx.y;
  const fa::MdItem& it = args.it[blockIdx.z];
  const int n = 1 << logn;
  const double q = pr[t].q, qinv = pr[t].qinv, pv = pr[t].pinv;
  const size_t o = (size_t)t * n;
  FinishSt st{it.uQ + o, it.base ? it.base + o : nullptr, it.out + o, it.gal, logn, q, qinv, pv, pv * qinv};
  const int H = 1 << (logn - 8);
  fwd_b_body(it.conv + o, st, twt + (size_t)t * 256, twr + (size_t)t * H * 8, q, qinv, logn, sm);
}

// ModDown finish of a rotation with its key-switch sum on the ciphertext
// primes formed in place: for limb t < L and the tile's words k,
//   u_h[k] = sum_i sigma(ext_i)[k] * key_i[h][t][k]   (h = 0, 1; own limbs from c1)
//   out0[k] = c0[pi(k)] + b0[k] + (u_0[k] - conv0^[k]) * P^-1   (b0 = 0 for a rotation),
//   out1[k] = b1[k] + (u_1[k] - conv1^[k]) * P^-1       (b1 = 0 for a rotation)
// where conv_h^ is the forward transform of Conv_{P->Q} finished here (pass B).
// The sums never reach HBM; both polynomials of the rotation share one gather.
struct MdKsArgs {
  fa::MdKsItem it[FA_MAXMD];
};

// Work item decode shared by the key-switch kernels: `rest` runs over (x, y,
// key group) with x fastest; the nq items of a key group (the same rotation
// for nq queries, items g*nq .. g*nq+nq-1) use the same key words.  With
// nq > 1 the ids are decoded so that those nq workgroups run one after the
// other on one XCD (ids 8 apart) and share the key words in its L2.  Returns
// false for the padding ids of the last group of eight.
__device__ __forceinline__ bool ks_decode(unsigned W, int nx, int ny, int nq, int ngroup, int& x, int& y, int& item) {
  unsigned rest = W, qi = 0;
  if (nq > 1) {
    const unsigned j8 = W >> 3;
    qi = j8 % (unsigned)nq;
    rest = (j8 / (unsigned)nq) * 8u + (W & 7u);
  }
  if (rest >= (unsigned)(nx * ny * ngroup)) return false;
  x = (int)(rest % (unsigned)nx);
  y = (int)((rest / (unsigned)nx) % (unsigned)ny);
  item = (int)(rest / (unsigned)(nx * ny)) * nq + (int)qi;
  return true;
}

// One query's key switches (nq == 1): ids decoded source-tile-major with the
// items fastest within an XCD, so the workgroups one XCD runs back to back (ids
// 8 apart) take the same source tile x of prime y for every rotation of the
// launch; the digits and c0 words of that tile, which every rotation gathers
// (through its own automorphism, into its own output tile), are read from HBM
// once and from that XCD's L2 after.  Returns false for the padding ids.
__device__ __forceinline__ bool ks_decode_src(unsigned W, int nx, int ny, int m, int& x, int& y, int& item) {
  const unsigned j8 = W >> 3;
  item = (int)(j8 % (unsigned)m);
  const unsigned rest = (j8 / (unsigned)m) * 8u + (W & 7u);
  if (rest >= (unsigned)(nx * ny)) return false;
  x = (int)(rest % (unsigned)nx);
  y = (int)(rest / (unsigned)nx);
  return true;
}

template <int DNUM, int ROWS, bool NT>
__global__ __launch_bounds__(256) void k_moddown_ks_b(MdKsArgs args, const DevPrime* __restrict__ pr,
                                                      const double* __restrict__ twt, const double* __restrict__ twr,
                                                      int logn, int L, int np, int alpha, int nq, int ngroup) {
  __shared__ double sm[ROWS * ROWW];
  const int n = 1 << logn;
  int tile, t, item;
  if (nq == 1) {
    int src;
    if (!ks_decode_src(blockIdx.x, (n >> 8) / ROWS, L, ngroup, src, t, item)) return;
    // the output tile whose automorphism image is the source tile
    tile = (int)(perm((uint32_t)src * (ROWS * 256u), args.it[item].inv_gal, logn) / (ROWS * 256u));
  } else if (!ks_decode(blockIdx.x, (n >> 8) / ROWS, L, nq, ngroup, tile, t, item)) {
    return;
  }
  const fa::MdKsItem& it = args.it[item];
  const int row0 = tile * ROWS;
  const uint32_t k0 = (uint32_t)row0 * 256u + threadIdx.x;  // this thread's words: k0 + 256 j, j < ROWS
  const double q = pr[t].q, qinv = pr[t].qinv, pv = pr[t].pinv, pvp = pv * qinv;
  const int own = t / alpha;
  const double* __restrict__ T = twt + (size_t)t * 256;
  const double* __restrict__ F = twr + (size_t)t * (n >> 8) * 8;
  const size_t o = (size_t)t * n;
  double u0[ROWS], u1[ROWS];
#pragma unroll
  for (int j = 0; j < ROWS; ++j) u0[j] = u1[j] = 0.0;
#pragma unroll 1
  for (int i = 0; i < DNUM; ++i) {
    const double* __restrict__ src = i == own ? it.c1 + o : it.ext + ((size_t)i * np + t) * n;
    const double* __restrict__ kb = it.key + (((size_t)i * 2 + 0) * np + t) * n + k0;
    const double* __restrict__ ka = it.key + (((size_t)i * 2 + 1) * np + t) * n + k0;
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
      const double x = src[perm(k0 + 256u * j, it.gal, logn)];
      // NT (one query): each key word is used once, so it streams past the
      // caches; several queries share it through L2 (see ks_decode)
      const double b = NT ? __builtin_nontemporal_load(kb + 256 * j) : kb[256 * j];
      const double a = NT ? __builtin_nontemporal_load(ka + 256 * j) : ka[256 * j];
      u0[j] += mul(x, b, q, qinv);
      u1[j] += mul(x, a, q, qinv);
    }
  }
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    u0[j] = reduce(u0[j], q, qinv);
    u1[j] = reduce(u1[j], q, qinv);
  }
  fwd_b_lds(it.conv + o, row0, ROWS, T, F, q, qinv, sm);
  double c0[ROWS];  // all loads before the first store, which may alias them for all the compiler knows
#pragma unroll
  for (int j = 0; j < ROWS; ++j) c0[j] = it.c0[o + perm(k0 + 256u * j, it.gal, logn)];
  if (it.b0) {
#pragma unroll
    for (int j = 0; j < ROWS; ++j) c0[j] += it.b0[o + k0 + 256 * j];
  }
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const int e = threadIdx.x + 256 * j;
    const double r = mulc(u0[j] - sm[lds_row(e >> 8, e & 255)], pv, pvp, q) + c0[j];
    __builtin_nontemporal_store(canon_full(r, q, qinv), it.out + o + k0 + 256 * j);
  }
  __syncthreads();
  fwd_b_lds(it.conv + (size_t)L * n + o, row0, ROWS, T, F, q, qinv, sm);
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const int e = threadIdx.x + 256 * j;
    double r = mulc(u1[j] - sm[lds_row(e >> 8, e & 255)], pv, pvp, q);
    if (it.b1) r += it.b1[o + k0 + 256 * j];
    __builtin_nontemporal_store(canon_full(r, q, qinv), it.out + (size_t)L * n + o + k0 + 256 * j);
  }
}

// Inverse pass B (the first pass of the inverse transform) of the 16 rows of sm
// (lds_row layout, canonical words, synchronised) into a: a thread transforms 16
// consecutive words, then 16 words 16 apart.  The rows come through LDS because
// 16 consecutive words a lane straight from memory are 64 lines an instruction.
__device__ __forceinline__ void inv_b_rows(double* sm, double* __restrict__ a, int row0, const double* __restrict__ T,
                                           const double* __restrict__ F, double q, double qinv) {
  const int l = threadIdx.x & 15, rl = threadIdx.x >> 4, r = row0 + rl;
  double x[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) x[m] = sm[lds_row(rl, 16 * l + m)];
#pragma unroll
  for (int s1 = 7; s1 >= 4; --s1) {
    const int half = 8 >> (s1 - 4);
    const double f = F[r * 8 + s1];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      if (m & half) continue;
      const double w = twb(T, f, s1, (l << (s1 - 4)) + (m >> (8 - s1)), q, qinv);
      if (s1 >= 6) gs_bfly<false>(x[m], x[m + half], w, q, qinv);
      else gs_bfly<true>(x[m], x[m + half], w, q, qinv);
    }
  }
#pragma unroll
  for (int m = 0; m < 16; ++m) sm[lds_row(rl, 16 * l + m)] = x[m];
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 16; ++m) x[m] = sm[lds_row(rl, l + 16 * m)];
#pragma unroll
  for (int s1 = 3; s1 >= 0; --s1) {
    const int half = 8 >> s1;
    const double f = F[r * 8 + s1];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      if (m & half) continue;
      gs_bfly(x[m], x[m + half], twb(T, f, s1, m >> (4 - s1), q, qinv), q, qinv);
    }
  }
#pragma unroll
  for (int m = 0; m < 16; ++m) a[(size_t)r * 256 + l + 16 * m] = x[m];
}

// src -> ptr
__global__ __launch_bounds__(256) void k_ntt_inv_b(LimbList ll, const DevPrime* __restrict__ pr,
                                                   const double* __restrict__ twt, const double* __restrict__ twr,
                                                   int logn) {
  __shared__ double sm[16 * ROWW];
  const int row0 = blockIdx.x * 16;
  const int pi = ll.prime[blockIdx.y];
  const double q = pr[pi].q, qinv = pr[pi].qinv;
  const double* __restrict__ src = ll.src[blockIdx.y] + (size_t)row0 * 256 + threadIdx.x;
  double x[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) x[j] = src[256 * j];
#pragma unroll
  for (int j = 0; j < 16; ++j) sm[lds_row(j, threadIdx.x)] = x[j];
  __syncthreads();
  inv_b_rows(sm, ll.ptr[blockIdx.y], row0, twt + (size_t)pi * 256, twr + (size_t)pi * (1 << logn >> 8) * 8, q, qinv);
}

// ---------------------------------------------------------------------------
// key-switch inner product on the special primes with the automorphism folded
// into the read of the extended digits
// ---------------------------------------------------------------------------
#define FA_MAXKS 32
struct KsArgs {
  fa::KsItem it[FA_MAXKS];
};

template <int DNUM>
__global__ __launch_bounds__(256) void k_ks_inner(KsArgs args, const DevPrime* __restrict__ pr, int logn, int L,
                                                  int np, int nq, int ngroup) {
  const int n = 1 << logn, K = np - L;
  int kx, tr, item;
  if (nq == 1) {
    int src;
    if (!ks_decode_src(blockIdx.x, n / 256, K, ngroup, src, tr, item)) return;
    kx = (int)(perm((uint32_t)src * 256u, args.it[item].inv_gal, logn) / 256u);  // see k_moddown_ks_b
  } else if (!ks_decode(blockIdx.x, n / 256, K, nq, ngroup, kx, tr, item)) {
    return;
  }
  const int k = kx * 256 + threadIdx.x;
  const int t = L + tr;
  const fa::KsItem& it = args.it[item];
  const double q = pr[t].q, qinv = pr[t].qinv;
  const uint32_t kk = perm((uint32_t)k, it.gal, logn);
  double x[DNUM], kb[DNUM], ka[DNUM];
#pragma unroll
  for (int i = 0; i < DNUM; ++i) {
    x[i] = it.ext[((size_t)i * np + t) * n + kk];
    kb[i] = __builtin_nontemporal_load(it.key + (((size_t)i * 2 + 0) * np + t) * n + k);
    ka[i] = __builtin_nontemporal_load(it.key + (((size_t)i * 2 + 1) * np + t) * n + k);
  }
  double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
  for (int i = 0; i < DNUM; ++i) {
    acc0 += mul(x[i], kb[i], q, qinv);
    acc1 += mul(x[i], ka[i], q, qinv);
  }
  it.u[(size_t)tr * n + k] = canon_full(acc0, q, qinv);
  it.u[((size_t)K + tr) * n + k] = canon_full(acc1, q, qinv);
}

// Key-switch sum on the special primes fused with the first pass of its
// inverse transform: for special prime t and the workgroup's 16 rows,
//   u_h = sum_i sigma(ext_i) * key_i[h]   (h = 0, 1)
// formed with consecutive threads on consecutive words, each polynomial then
// through LDS and inverse pass B into it.u, in place of k_ks_inner's sums after
// k_ntt_inv_b.
template <int DNUM, bool NT>
__global__ __launch_bounds__(256) void k_ks_inv_b(KsArgs args, const DevPrime* __restrict__ pr,
                                                  const double* __restrict__ twt, const double* __restrict__ twr,
                                                  int logn, int L, int np, int nq, int ngroup) {
  __shared__ double sm[16 * ROWW];
  const int n = 1 << logn;
  int tile, tr, item;
  if (nq == 1) {
    int src;
    if (!ks_decode_src(blockIdx.x, n >> 12, np - L, ngroup, src, tr, item)) return;
    tile = (int)(perm((uint32_t)src << 12, args.it[item].inv_gal, logn) >> 12);
  } else if (!ks_decode(blockIdx.x, n >> 12, np - L, nq, ngroup, tile, tr, item)) {
    return;
  }
  const int t = L + tr;
  const fa::KsItem& it = args.it[item];
  const double q = pr[t].q, qinv = pr[t].qinv;
  const double* __restrict__ T = twt + (size_t)t * 256;
  const double* __restrict__ F = twr + (size_t)t * (n >> 8) * 8;
  const uint32_t k0 = ((uint32_t)tile << 12) + threadIdx.x;  // this thread's words: k0 + 256 j
  double y0[16], y1[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) y0[j] = y1[j] = 0.0;
#pragma unroll 1
  for (int i = 0; i < DNUM; ++i) {
    const double* __restrict__ src = it.ext + ((size_t)i * np + t) * n;
    const double* __restrict__ kb = it.key + (((size_t)i * 2 + 0) * np + t) * n + k0;
    const double* __restrict__ ka = it.key + (((size_t)i * 2 + 1) * np + t) * n + k0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const double x = src[perm(k0 + 256u * j, it.gal, logn)];
      const double b = NT ? __builtin_nontemporal_load(kb + 256 * j) : kb[256 * j];
      const double a = NT ? __builtin_nontemporal_load(ka + 256 * j) : ka[256 * j];
      y0[j] += mul(x, b, q, qinv);
      y1[j] += mul(x, a, q, qinv);
    }
  }
  double* out = it.u + (size_t)tr * n;
#pragma unroll
  for (int j = 0; j < 16; ++j) sm[lds_row(j, threadIdx.x)] = reduce(y0[j], q, qinv);
  __syncthreads();
  inv_b_rows(sm, out, tile * 16, T, F, q, qinv);
  __syncthreads();  // the second polynomial reuses the LDS rows
#pragma unroll
  for (int j = 0; j < 16; ++j) sm[lds_row(j, threadIdx.x)] = reduce(y1[j], q, qinv);
  __syncthreads();
  inv_b_rows(sm, out + (size_t)(np - L) * n, tile * 16, T, F, q, qinv);
}

// ---------------------------------------------------------------------------
// Giant steps of the diagonal scoring, fused: for every block and every
// ciphertext/special prime t,
//   u[blk] = sum_{g=1}^{G-1} ( sum_i sigma_g(ext[blk][g]_i) * key_g[i]  +  P * sigma_g(acc_g.c0) )
// where ext holds the first forward pass only of the extended digits of
// acc_g.c1.  A workgroup owns one tile of rows*256 output words of one prime:
// for each (g, digit) it runs the last eight NTT stages on the source tile
// (the automorphism maps an aligned tile onto an aligned tile) in LDS, then
// gathers through the permutation and multiplies by the key, so the digits in
// NTT form never reach HBM.  The digit's own limbs come from acc_g.c1 itself.
// Workgroup ids are decoded so that the nb blocks of one (tile, prime) land on
// the same XCD one after the other and share the key rows in its L2.
//
// A workgroup is a serial chain of giants times digits, each a load, two halves
// of a row pass and a gather with barriers between: 7.5 us apiece whatever else
// runs.  Where the (tile, prime, block) triples leave the chip's 512 places (two
// workgroups a CU) more than half empty, the giants are split into groups with
// sums of their own, added by k_sum_parts: one block at N = 2^16 and 12+3 primes
// (240 triples, 7 giants) took 210 us in one group.  The parts lie in the ModUps'
// scratch, which bounds them too: it holds giants / blocks * L / (L + K) parts with
// the default two lanes (half of that with one), none from blocks >= giants on.
// ---------------------------------------------------------------------------
#define FA_MAXG 32
struct GiantArgs {
  const double* ext;  // [nb][ng][dnum][np][N], first pass only
  const double* acc;  // acc of block blk, giant g: acc + blk * astride + g * 2 L N
  const double* key[FA_MAXG];
  uint32_t gal[FA_MAXG];
  double* u;          // [nb][2][np][N]
  double* part;       // sums of the giant groups after the first, each as u
  size_t astride;
  int nb, ng, ngs, g0, accumulate;  // ng giants in this launch; ngs: the giant stride of ext
  int per;                          // giants per group (blockIdx.y)
};

template <int DNUM, int ROWS>
__global__ __launch_bounds__(256) void k_giant_ks(GiantArgs a, const DevPrime* __restrict__ pr,
                                                  const double* __restrict__ twt, const double* __restrict__ twr,
                                                  int logn, int L, int np, int alpha, int ntile) {
  __shared__ double sm[ROWS * ROWW];
  const unsigned W = blockIdx.x;
  const unsigned j8 = W >> 3;
  const int blk = (int)(j8 % (unsigned)a.nb);
  const unsigned rest = (j8 / (unsigned)a.nb) * 8u + (W & 7u);
  if (rest >= (unsigned)(ntile * np)) return;
  const int t = (int)(rest / (unsigned)ntile), tile = (int)(rest % (unsigned)ntile);
  const int n = 1 << logn;
  constexpr uint32_t TW = ROWS * 256u;  // words of a tile; ROWS words per thread
  const uint32_t k0 = (uint32_t)tile * TW;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const double* __restrict__ T = twt + (size_t)t * 256;
  const double* __restrict__ F = twr + (size_t)t * (n >> 8) * 8;
  const int own = t < L ? t / alpha : -1;
  const size_t ln = (size_t)L * n;
  double acc0[ROWS], acc1[ROWS];
#pragma unroll
  for (int j = 0; j < ROWS; ++j) acc0[j] = acc1[j] = 0.0;
  const int glo = (int)blockIdx.y * a.per, ghi = min(a.ng, glo + a.per);
#pragma unroll 1
  for (int g = glo; g < ghi; ++g) {
    const uint32_t gal = a.gal[g];
    const uint32_t sbase = perm(k0, gal, logn) & ~(TW - 1u);
    const double* __restrict__ accg = a.acc + (size_t)blk * a.astride + (size_t)(a.g0 + g) * 2 * ln;
    const double* __restrict__ key = a.key[g];
#pragma unroll 1
    for (int i = 0; i < DNUM; ++i) {
      // opaque copies: recomputing the permutation per digit is cheaper than
      // keeping it (and the twiddle loads) live across the loop
      uint32_t galv = gal;
      const double* Tv = T;
      asm volatile("" : "+s"(galv), "+s"(Tv));
      const double* __restrict__ kb = key + (((size_t)i * 2 + 0) * np + t) * n + k0 + threadIdx.x;
      const double* __restrict__ ka = key + (((size_t)i * 2 + 1) * np + t) * n + k0 + threadIdx.x;
      double x[ROWS];
      if (i == own) {
        const double* __restrict__ c1 = accg + ln + (size_t)t * n;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) x[j] = c1[perm(k0 + threadIdx.x + 256u * j, galv, logn)];
      } else {
        const double* src = a.ext + ((((size_t)blk * a.ngs + g) * DNUM + i) * np + t) * n;
        fwd_b_lds(src, (int)(sbase >> 8), ROWS, Tv, F, q, qinv, sm);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
          const uint32_t sk = perm(k0 + threadIdx.x + 256u * j, galv, logn) - sbase;
          x[j] = sm[lds_row((int)(sk >> 8), (int)(sk & 255u))];
        }
        __syncthreads();  // the next digit's pass reuses the LDS tile
      }
      add_digit<DNUM>(acc0, acc1, x, kb, ka, 256, i, q, qinv);
    }
    if (t < L) {
      const double* __restrict__ c0 = accg + (size_t)t * n;
      const double pm = pr[t].pmod;
#pragma unroll
      for (int j = 0; j < ROWS; ++j) acc0[j] += mul(c0[perm(k0 + threadIdx.x + 256u * j, gal, logn)], pm, q, qinv);
    }
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
      acc0[j] = reduce(acc0[j], q, qinv);
      acc1[j] = reduce(acc1[j], q, qinv);
    }
  }
  double* u = blockIdx.y ? a.part + (size_t)(blockIdx.y - 1) * a.nb * 2 * np * n : a.u;
  double* u0 = u + ((size_t)blk * 2 * np + t) * n + k0 + threadIdx.x;
  double* u1 = u0 + (size_t)np * n;
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    double r0 = acc0[j], r1 = acc1[j];
    if (a.accumulate) {
      r0 += u0[256 * j];
      r1 += u1[256 * j];
    }
    u0[256 * j] = canon_full(r0, q, qinv);
    u1[256 * j] = canon_full(r1, q, qinv);
  }
}

// u += the parts parts of `words` words each, canonical (limb r over prime r % np)
__global__ __launch_bounds__(256) void k_sum_parts(double* __restrict__ u, const double* __restrict__ part, int parts,
                                                   const DevPrime* __restrict__ pr, int logn, int np) {
  const size_t o = ((size_t)blockIdx.y << logn) + blockIdx.x * 256 + threadIdx.x;
  const size_t words = (size_t)gridDim.y << logn;
  const int t = blockIdx.y % np;
  double v = u[o];
  for (int i = 0; i < parts; ++i) v += part[i * words + o];  // at most 7 parts: below 8q
  u[o] = canon_full(v, pr[t].q, pr[t].qinv);
}

// ---------------------------------------------------------------------------
// diagonal-layout multiply-accumulate: the HBM stream of the scoring path
//   acc_j[pair][h][t][k] = sum_b pts[blk][g*B+b][t][k] * qrot_j[b][h][t][k]
// for NQ queries j at once, pair = (blk, g).  Each wave owns 64 consecutive
// coefficients and keeps NACC pairs x NQ queries x 2 accumulators in
// registers; every plaintext word is read once per group of NQ queries.
//
// The operands of a step (NACC plaintext words and each query's two rotated
// words per coefficient) travel HBM -> LDS with direct-to-LDS loads into a
// ring of S per-wave slots: while step b is multiplied out of LDS, steps
// b+1..b+S-1 are in flight, and they occupy no registers.  A wave only reads
// its own slots, so the vector-memory counter (loads complete in order) is
// the only synchronisation: before step b, wait until at most the loads of
// the later steps are outstanding.  A reduction every 8 products keeps the
// lazy sums below 2^53.
//
// With several chunks of NACC pairs in one launch, workgroup ids are decoded
// so that the chunks of one coefficient tile run on one XCD back to back and
// read the rotated queries from that XCD's L2 after the first.
// ---------------------------------------------------------------------------
#define FA_MAXBLK 32
struct MacArgs {
  const double* q0[FA_MAXQ];    // per query: rotation 0 (the query itself)
  const double* qrot[FA_MAXQ];  // per query: rotations 1..B-1, [B-1][2][L][N]
  double* acc[FA_MAXQ];         // per query: [n_pairs][2][L][N]
  const double* blk[FA_MAXBLK];
  int n_pairs, pair0, B, logG, L;
  int nchunk, ntile;            // chunks of NACC pairs from pair0; tiles of 256 words
};

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void gbl_void_t;

// s_waitcnt immediate (gfx9 encoding): wait until at most n vector-memory
// operations are outstanding; the LDS and export counters are not waited on
#define FA_VMCNT(n) (0x0F70 | ((n) & 15) | (((n) >> 4) << 14))
#define FA_LGKMCNT0 0xC07F

template <int NQ, int NACC, int S>
__global__ __launch_bounds__(256) void k_mac_diag(MacArgs args, const DevPrime* __restrict__ pr, int logn) {
  constexpr int ROWS = NACC + 2 * NQ;    // 64-word rows of one step: plaintexts, then x0/x1 per query
  constexpr int GL = NACC / 2 + NQ;      // loads issued per step
  static_assert(S == 2 || S == 3, "ring of two or three slots");
  static_assert((S - 1) * GL <= 63, "vector-memory counter range");
  __shared__ double slab[4][S][ROWS][64];
  unsigned tile = blockIdx.x, chunk = 0;
  if (args.nchunk > 1) {
    const unsigned j = blockIdx.x >> 3;
    chunk = j % (unsigned)args.nchunk;
    tile = (j / (unsigned)args.nchunk) * 8u + (blockIdx.x & 7u);
    if (tile >= (unsigned)args.ntile) return;
  }
  const int n = 1 << logn;
  const size_t ln = (size_t)args.L * n;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const size_t c0 = (size_t)tile * 256 + (size_t)w * 64;  // first coefficient of this wave
  const size_t f = c0 + lane;
  const int t = (int)(c0 >> logn);
  const double q = pr[t].q, qinv = pr[t].qinv;
  const int pair0 = args.pair0 + (int)chunk * NACC;
  const int last = args.n_pairs - 1;
  const int G = 1 << args.logG;
  const int B = args.B;
  const int hp = lane >> 5;                         // which of the two rows a lane's 16 bytes land in
  const size_t lo = c0 + 2 * (size_t)(lane & 31);   // its two coefficients
  // per-lane source of each load at step 0 (step b adds b * ln words): lanes
  // 0-31 read pair 2i, lanes 32-63 pair 2i+1 (pairs past the end re-read the
  // last pair, in bounds, and are never stored); the queries' x0 / x1 rows
  const double* src[NACC / 2];
#pragma unroll
  for (int i = 0; i < NACC / 2; ++i) {
    const int pa = min(pair0 + 2 * i, last), pb = min(pair0 + 2 * i + 1, last);
    const double* xa = args.blk[pa >> args.logG] + (size_t)((pa & (G - 1)) * B) * ln;
    const double* xb = args.blk[pb >> args.logG] + (size_t)((pb & (G - 1)) * B) * ln;
    src[i] = (hp ? xb : xa) + lo;
  }
  const double* qs0[NQ];
  const double* qsr[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    qs0[j] = args.q0[j] + (size_t)hp * ln + lo;
    qsr[j] = args.qrot[j] + (size_t)hp * ln + lo;
  }
  // one step's loads into slot sl: row 2i gets pair 2i, row 2i+1 pair 2i+1
  auto issue = [&](int sl, int b) {
#pragma unroll
    for (int i = 0; i < NACC / 2; ++i)
      __builtin_amdgcn_global_load_lds((gbl_void_t*)(src[i] + (size_t)b * ln), (lds_void_t*)&slab[w][sl][2 * i][0],
                                       16, 0, 0);
#pragma unroll
    for (int j = 0; j < NQ; ++j)
      __builtin_amdgcn_global_load_lds((gbl_void_t*)(b == 0 ? qs0[j] : qsr[j] + (size_t)(b - 1) * 2 * ln),
                                       (lds_void_t*)&slab[w][sl][NACC + 2 * j][0], 16, 0, 0);
  };
  double* accp[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j) accp[j] = args.acc[j];
  const int cnt = min(NACC, args.n_pairs - pair0);
  double a0[NQ][NACC], a1[NQ][NACC];
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int i = 0; i < NACC; ++i) {
      a0[j][i] = 0.0;
      a1[j][i] = 0.0;
    }
#pragma unroll
  for (int sl = 0; sl < S; ++sl)
    if (sl < B) issue(sl, sl);
  // one step out of slot SL (a compile-time slot index lets the compiler's
  // tracking of pending direct-to-LDS loads tell the slots apart)
  auto step = [&](auto slc, int b) {
    constexpr int SL = decltype(slc)::value;
    // steps b+1 .. min(b+S-1, B-1) were issued after step b
    const int later = min(S - 1, B - 1 - b);
    __builtin_amdgcn_sched_barrier(0);
    if (later >= 2) __builtin_amdgcn_s_waitcnt(FA_VMCNT(2 * GL));
    else if (later == 1) __builtin_amdgcn_s_waitcnt(FA_VMCNT(GL));
    else __builtin_amdgcn_s_waitcnt(FA_VMCNT(0));
    __builtin_amdgcn_sched_barrier(0);
    double x0[NQ], x1[NQ], x0p[NQ], x1p[NQ];
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      x0[j] = slab[w][SL][NACC + 2 * j][lane];
      x1[j] = slab[w][SL][NACC + 2 * j + 1][lane];
      x0p[j] = x0[j] * qinv;
      x1p[j] = x1[j] * qinv;
    }
#pragma unroll
    for (int i0 = 0; i0 < NACC; i0 += 8) {
      double p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) p[i] = slab[w][SL][i0 + i][lane];
#pragma unroll
      for (int j = 0; j < NQ; ++j)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          a0[j][i0 + i] += mulc(p[i], x0[j], x0p[j], q);
          a1[j][i0 + i] += mulc(p[i], x1[j], x1p[j], q);
        }
    }
    if ((b & 7) == 7) {
#pragma unroll
      for (int j = 0; j < NQ; ++j)
#pragma unroll
        for (int i = 0; i < NACC; ++i) {
          a0[j][i] = reduce(a0[j][i], q, qinv);
          a1[j][i] = reduce(a1[j][i], q, qinv);
        }
    }
    // the slot is read out: refill it with step b+S
    __builtin_amdgcn_s_waitcnt(FA_LGKMCNT0);
    __builtin_amdgcn_sched_barrier(0);
    if (b + S < B) issue(SL, b + S);
  };
  for (int b0 = 0; b0 < B; b0 += S) {
    step(std::integral_constant<int, 0>{}, b0);
    if (b0 + 1 < B) step(std::integral_constant<int, 1>{}, b0 + 1);
    if constexpr (S > 2)
      if (b0 + 2 < B) step(std::integral_constant<int, 2>{}, b0 + 2);
  }
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int i = 0; i < NACC; ++i) {
      if (i < cnt) {
        double* o = accp[j] + (size_t)(pair0 + i) * 2 * ln + f;
        o[0] = canon_full(a0[j][i], q, qinv);
        o[ln] = canon_full(a1[j][i], q, qinv);
      }
    }
}

// One query, NACC pairs: the same product with three steps in flight per wave.
// Steps cycle through two LDS slots (direct-to-LDS loads of the NACC plaintext
// rows, the rotated query in registers) and one register stage (the NACC
// plaintext words and the rotated query loaded straight into registers), so a
// wave holds the loads of three steps while it multiplies one.  The LDS
// slots are synchronised by the vector-memory counter as in k_mac_diag (a
// slot's wait counts the loads issued after it); the register stage is waited
// on by the compiler.  Reductions every 6 steps (lazy sums below 6q + q/2).
template <int NACC>
__global__ __launch_bounds__(256) void k_mac_diag3(MacArgs args, const DevPrime* __restrict__ pr, int logn) {
  constexpr int ROWS = NACC + 2;    // an LDS step: the plaintext rows, then the rotated query's x0 / x1
  constexpr int GL = NACC / 2 + 1;  // vector-memory operations of an LDS step
  constexpr int GR = NACC + 2;      // of a register step
  static_assert(GL + GR <= 63, "vector-memory counter range");
  __shared__ double slab[4][2][ROWS][64];
  unsigned tile = blockIdx.x, chunk = 0;
  if (args.nchunk > 1) {
    const unsigned j = blockIdx.x >> 3;
    chunk = j % (unsigned)args.nchunk;
    tile = (j / (unsigned)args.nchunk) * 8u + (blockIdx.x & 7u);
    if (tile >= (unsigned)args.ntile) return;
  }
  const int n = 1 << logn;
  const size_t ln = (size_t)args.L * n;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const size_t c0 = (size_t)tile * 256 + (size_t)w * 64;
  const size_t f = c0 + lane;
  const int t = (int)(c0 >> logn);
  const double q = pr[t].q, qinv = pr[t].qinv;
  const int pair0 = args.pair0 + (int)chunk * NACC;
  const int last = args.n_pairs - 1;
  const int G = 1 << args.logG;
  const int B = args.B;
  const int hp = lane >> 5;
  const size_t lo = c0 + 2 * (size_t)(lane & 31);
  // plaintext row of pair i at step 0 (pairs past the end re-read the last pair)
  auto row = [&](int i) -> const double* {
    const int pa = min(pair0 + i, last);
    return args.blk[pa >> args.logG] + (size_t)((pa & (G - 1)) * B) * ln;
  };
  const double* src[NACC / 2];  // direct-to-LDS source of load i (pairs 2i, 2i+1)
#pragma unroll
  for (int i = 0; i < NACC / 2; ++i) src[i] = (hp ? row(2 * i + 1) : row(2 * i)) + lo;
  const double* qd0 = args.q0[0] + (size_t)hp * ln + lo;    // direct-to-LDS: x0 row (lanes 0-31), x1 row
  const double* qdr = args.qrot[0] + (size_t)hp * ln + lo;
  const double* qv0 = args.q0[0] + f;                       // into registers
  const double* qvr = args.qrot[0] + f;
  double a0[NACC], a1[NACC];
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    a0[i] = 0.0;
    a1[i] = 0.0;
  }
  auto dma = [&](auto slc, int b) {
    constexpr int SL = decltype(slc)::value;
#pragma unroll
    for (int i = 0; i < NACC / 2; ++i)
      __builtin_amdgcn_global_load_lds((gbl_void_t*)(src[i] + (size_t)b * ln), (lds_void_t*)&slab[w][SL][2 * i][0],
                                       16, 0, 0);
    __builtin_amdgcn_global_load_lds((gbl_void_t*)(b == 0 ? qd0 : qdr + (size_t)(b - 1) * 2 * ln),
                                     (lds_void_t*)&slab[w][SL][NACC][0], 16, 0, 0);
  };
  double pv[NACC], xr0, xr1;
  auto rld = [&](int b) {
#pragma unroll
    for (int i = 0; i < NACC; ++i) pv[i] = __builtin_nontemporal_load(row(i) + (size_t)b * ln + f);
    const double* x = b == 0 ? qv0 : qvr + (size_t)(b - 1) * 2 * ln;
    xr0 = x[0];
    xr1 = x[ln];
  };
  auto mac_lds = [&](auto slc) {
    constexpr int SL = decltype(slc)::value;
    const double x0 = slab[w][SL][NACC][lane], x1 = slab[w][SL][NACC + 1][lane];
    const double x0p = x0 * qinv, x1p = x1 * qinv;
#pragma unroll
    for (int c = 0; c < NACC; c += 8) {
      double pc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) pc[i] = slab[w][SL][c + i][lane];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        a0[c + i] += mulc(pc[i], x0, x0p, q);
        a1[c + i] += mulc(pc[i], x1, x1p, q);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  dma(S0{}, 0);
  if (B > 1) dma(S1{}, 1);
  if (B > 2) rld(2);
  int red = 0;
  for (int b = 0; b < B; b += 3) {
    // step b out of slot 0: issued after its loads are slot 1's step (if any)
    // and the register step (if any), in that order
    __builtin_amdgcn_sched_barrier(0);
    if (b + 2 < B) __builtin_amdgcn_s_waitcnt(FA_VMCNT(GL + GR));
    else if (b + 1 < B) __builtin_amdgcn_s_waitcnt(FA_VMCNT(GL));
    else __builtin_amdgcn_s_waitcnt(FA_VMCNT(0));
    __builtin_amdgcn_sched_barrier(0);
    mac_lds(S0{});
    __builtin_amdgcn_s_waitcnt(FA_LGKMCNT0);
    __builtin_amdgcn_sched_barrier(0);
    const bool n0 = b + 3 < B, n1 = b + 4 < B, n2 = b + 5 < B;
    if (n0) dma(S0{}, b + 3);
    if (b + 1 < B) {
      // step b+1 out of slot 1: issued after it are the register step (when
      // b+2 < B) and slot 0's refill (when b+3 < B)
      __builtin_amdgcn_sched_barrier(0);
      if (n0) __builtin_amdgcn_s_waitcnt(FA_VMCNT(GR + GL));
      else if (b + 2 < B) __builtin_amdgcn_s_waitcnt(FA_VMCNT(GR));
      else __builtin_amdgcn_s_waitcnt(FA_VMCNT(0));
      __builtin_amdgcn_sched_barrier(0);
      mac_lds(S1{});
      __builtin_amdgcn_s_waitcnt(FA_LGKMCNT0);
      __builtin_amdgcn_sched_barrier(0);
      if (n1) dma(S1{}, b + 4);
    }
    if (b + 2 < B) {
      // step b+2 out of registers (the compiler waits for them)
      const double x0p = xr0 * qinv, x1p = xr1 * qinv;
#pragma unroll
      for (int i = 0; i < NACC; ++i) {
        a0[i] += mulc(pv[i], xr0, x0p, q);
        a1[i] += mulc(pv[i], xr1, x1p, q);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (n2) rld(b + 5);
    }
    if (++red == 2) {
      red = 0;
#pragma unroll
      for (int i = 0; i < NACC; ++i) {
        a0[i] = reduce(a0[i], q, qinv);
        a1[i] = reduce(a1[i], q, qinv);
      }
    }
  }
  const int cnt = min(NACC, args.n_pairs - pair0);
  double* accp = args.acc[0];
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    if (i < cnt) {
      double* o = accp + (size_t)(pair0 + i) * 2 * ln + f;
      o[0] = canon_full(a0[i], q, qinv);
      o[ln] = canon_full(a1[i], q, qinv);
    }
  }
}

// ---------------------------------------------------------------------------
// multiply-accumulate against an encrypted block (ct x ct, three components)
//   acc[pair][0] += c0 q0,  acc[pair][1] += c0 q1 + c1 q0,  acc[pair][2] += c1 q1
// with (c0, c1) = ct[blk][g*B+b] and (q0, q1) = rot_b.  One thread per
// coefficient, NACC pairs per chunk; several chunks in one launch share the
// rotated query through one XCD's L2 as in k_mac_diag.  A reduction every 4
// steps keeps the lazy sums below 2^53 (the middle component gains two
// products per step).
// ---------------------------------------------------------------------------
struct MacCtArgs {
  const double* q0;
  const double* qrot;
  double* acc;  // [n_pairs][3][L][N]
  const double* blk[FA_MAXBLK];
  int n_pairs, pair0, B, logG, L;
  int nchunk, ntile;
};

template <int NACC>
__global__ __launch_bounds__(256) void k_mac_diag_ct(MacCtArgs args, const DevPrime* __restrict__ pr, int logn) {
  unsigned tile = blockIdx.x, chunk = 0;
  if (args.nchunk > 1) {
    const unsigned j = blockIdx.x >> 3;
    chunk = j % (unsigned)args.nchunk;
    tile = (j / (unsigned)args.nchunk) * 8u + (blockIdx.x & 7u);
    if (tile >= (unsigned)args.ntile) return;
  }
  const int n = 1 << logn;
  const size_t ln = (size_t)args.L * n;
  const size_t f = (size_t)tile * 256 + threadIdx.x;
  const int t = (int)(f >> logn);
  const double q = pr[t].q, qinv = pr[t].qinv;
  const int pair0 = args.pair0 + (int)chunk * NACC;
  const int last = args.n_pairs - 1;
  const int G = 1 << args.logG;
  const double* src[NACC];
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    const int pair = min(pair0 + i, last);
    src[i] = args.blk[pair >> args.logG] + (size_t)((pair & (G - 1)) * args.B) * 2 * ln + f;
  }
  double a0[NACC], a1[NACC], a2[NACC];
#pragma unroll
  for (int i = 0; i < NACC; ++i) a0[i] = a1[i] = a2[i] = 0.0;
  for (int b = 0; b < args.B; ++b) {
    const double* __restrict__ qb = b == 0 ? args.q0 : args.qrot + (size_t)(b - 1) * 2 * ln;
    const double x0 = qb[f], x1 = qb[ln + f];
    double p0[NACC], p1[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) {
      p0[i] = __builtin_nontemporal_load(src[i] + (size_t)b * 2 * ln);
      p1[i] = __builtin_nontemporal_load(src[i] + (size_t)b * 2 * ln + ln);
    }
    const double x0p = x0 * qinv, x1p = x1 * qinv;
#pragma unroll
    for (int i = 0; i < NACC; ++i) {
      a0[i] += mulc(p0[i], x0, x0p, q);
      a1[i] += mulc(p0[i], x1, x1p, q) + mulc(p1[i], x0, x0p, q);
      a2[i] += mulc(p1[i], x1, x1p, q);
    }
    if ((b & 3) == 3) {
#pragma unroll
      for (int i = 0; i < NACC; ++i) {
        a0[i] = reduce(a0[i], q, qinv);
        a1[i] = reduce(a1[i], q, qinv);
        a2[i] = reduce(a2[i], q, qinv);
      }
    }
  }
  const int cnt = min(NACC, args.n_pairs - pair0);
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    if (i < cnt) {
      double* o = args.acc + (size_t)(pair0 + i) * 3 * ln + f;
      o[0] = canon_full(a0[i], q, qinv);
      o[ln] = canon_full(a1[i], q, qinv);
      o[2 * ln] = canon_full(a2[i], q, qinv);
    }
  }
}

// ---------------------------------------------------------------------------
// small element-wise kernels
// ---------------------------------------------------------------------------
#define FA_MAXPT 32
struct PtArgs {
  const double* pt[FA_MAXPT];
};

__global__ __launch_bounds__(256) void k_mul_plain(const double* __restrict__ ct, PtArgs pts, double* out,
                                                   const DevPrime* __restrict__ pr, int logn, int L) {
  const int n = 1 << logn;
  const size_t ln = (size_t)L * n;
  const size_t f = (size_t)blockIdx.x * 256 + threadIdx.x;
  const int w = blockIdx.y;
  const int t = (int)(f >> logn);
  const double q = pr[t].q, qinv = pr[t].qinv;
  const double p = pts.pt[w][f];
  double* o = out + (size_t)w * 2 * ln;
  o[f] = canon(mul(ct[f], p, q, qinv), q);
  o[ln + f] = canon(mul(ct[ln + f], p, q, qinv), q);
}

__global__ __launch_bounds__(256) void k_add_limbs(double* __restrict__ dst, const double* __restrict__ src,
                                                   const DevPrime* __restrict__ pr, int logn, int period) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int row = blockIdx.y;
  const double q = pr[row % period].q;
  const size_t o = (size_t)row * n + k;
  dst[o] = canon(dst[o] + src[o], q);
}

// --- the membership path: rescale, ct x ct tensor, constants -------------
#define FA_MAXLIMB 16
struct ResArgs {
  double c[FA_MAXLIMB];   // per limb: q_last^-1 mod q_t (rescale) or a constant mod q_t
  double cp[FA_MAXLIMB];  // c * (1/q_t)
};
#define FA_MAXTERM 8
struct TensorList {
  const double* x[FA_MAXTERM];
  const double* y[FA_MAXTERM];
  int xL[FA_MAXTERM], yL[FA_MAXTERM];
};
struct ChebFixArgs {
  double c[FA_MAXTERM][FA_MAXLIMB];
  double cp[FA_MAXTERM][FA_MAXLIMB];
  int odd[FA_MAXTERM];
};
struct LinArgs {
  const double* x[FA_MAXTERM];
  int xL[FA_MAXTERM];
  double c[FA_MAXTERM][FA_MAXLIMB];
  double cp[FA_MAXTERM][FA_MAXLIMB];
  double c0[FA_MAXLIMB];
  int nterm, accumulate;
};
// Rescale, second pass: out[h][t] = (c[h][t] - lift^[h][t]) * q_last^-1 (NTT form),
// t < L-1, with lift's row pass finished here; c has L limbs per polynomial
struct RescaleSt {
  const double* ct;
  double* out;
  double q, qinv, c, cp;
  struct Op {
    double u;
  };
  __device__ Op load(size_t i) const { return {ct[i]}; }
  __device__ void operator()(size_t i, double x, Op o) const {
    out[i] = canon_full(mulc(o.u - x, c, cp, q), q, qinv);
  }
};
__global__ __launch_bounds__(256) void k_rescale_b(const double* __restrict__ ct, double* lift,
                                                   double* __restrict__ out, ResArgs a,
                                                   const DevPrime* __restrict__ pr, const double* __restrict__ twt,
                                                   const double* __restrict__ twr, int logn, int L) {
  __shared__ double sm[16 * ROWW];
  const int n = 1 << logn, H = 1 << (logn - 8), t = blockIdx.y;
  const size_t h = blockIdx.z;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = (h * (L - 1) + t) * n;
  fwd_b_body(lift + o, RescaleSt{ct + (h * L + t) * n, out + o, q, qinv, a.c[t], a.cp[t]}, twt + (size_t)t * 256,
             twr + (size_t)t * H * 8, q, qinv, logn, sm);
}
// out = (x0 y0, x0 y1 + x1 y0, x1 y1) over the L primes (NTT form)
// ciphertext j = blockIdx.z: x_j = x + j*sx with xL limbs per polynomial (its first L
// limbs read: the drop to L is free), likewise y; out_j = out + j*3LN
__global__ __launch_bounds__(256) void k_tensor(const double* __restrict__ x, const double* __restrict__ y,
                                                double* __restrict__ out, const DevPrime* __restrict__ pr, int logn,
                                                int L, int xL, int yL, size_t sx, size_t sy) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y;
  const size_t j = blockIdx.z;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = (size_t)t * n + k, ln = (size_t)L * n;
  x += j * sx;
  y += j * sy;
  out += j * 3 * ln;
  const double x0 = x[o], x1 = x[(size_t)xL * n + o], y0 = y[o], y1 = y[(size_t)yL * n + o];
  out[o] = canon_full(mul(x0, y0, q, qinv), q, qinv);
  out[ln + o] = canon_full(mul(x0, y1, q, qinv) + mul(x1, y0, q, qinv), q, qinv);
  out[2 * ln + o] = canon_full(mul(x1, y1, q, qinv), q, qinv);
}
// tensors of count ciphertext pairs given by pointer (pair j = blockIdx.z): x_j with
// xL[j] limbs per polynomial (its first L read), likewise y_j; out_j = out + j*3LN
__global__ __launch_bounds__(256) void k_tensor_list(TensorList a, double* __restrict__ out,
                                                     const DevPrime* __restrict__ pr, int logn, int L) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y, j = blockIdx.z;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = (size_t)t * n + k, ln = (size_t)L * n;
  const double* __restrict__ x = a.x[j];
  const double* __restrict__ y = a.y[j];
  const double x0 = x[o], x1 = x[(size_t)a.xL[j] * n + o], y0 = y[o], y1 = y[(size_t)a.yL[j] * n + o];
  out += (size_t)j * 3 * ln;
  out[o] = canon_full(mul(x0, y0, q, qinv), q, qinv);
  out[ln + o] = canon_full(mul(x0, y1, q, qinv) + mul(x1, y0, q, qinv), q, qinv);
  out[2 * ln + o] = canon_full(mul(x1, y1, q, qinv), q, qinv);
}
// Chebyshev products, in place over count ciphertexts (pair j = blockIdx.z >> 1,
// polynomial h = blockIdx.z & 1): p_j <- 2 p_j - c_j T1 (odd[j]; T1 with t1L limbs per
// polynomial, its first L read) or 2 p_j + c_j on polynomial 0 (even)
__global__ __launch_bounds__(256) void k_cheb_fix(double* __restrict__ prod, const double* __restrict__ t1,
                                                  ChebFixArgs a, const DevPrime* __restrict__ pr, int logn, int L,
                                                  int t1L) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y, j = blockIdx.z >> 1, h = blockIdx.z & 1;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = ((size_t)(2 * j + h) * L + t) * n + k;
  double v = prod[o];
  v = v + v;
  if (a.odd[j]) v -= mulc(t1[((size_t)h * t1L + t) * n + k], a.c[j][t], a.cp[j][t], q);
  else if (h == 0) v += a.c[j][t];
  prod[o] = canon_full(v, q, qinv);
}
// out = (accumulate ? out : 0) + sum_i x_i * c_i (+ c0 on polynomial 0), one ciphertext;
// x_i canonical with xL[i] limbs per polynomial (its first L read); a reduction after
// every four terms keeps the lazy sum below 5q
__global__ __launch_bounds__(256) void k_lincomb(double* __restrict__ out, LinArgs a, const DevPrime* __restrict__ pr,
                                                 int logn, int L) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y, h = blockIdx.z;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = ((size_t)h * L + t) * n + k;
  double v = a.accumulate ? out[o] : 0.0;
  for (int i = 0; i < a.nterm; ++i) {
    v += mulc(a.x[i][((size_t)h * a.xL[i] + t) * n + k], a.c[i][t], a.cp[i][t], q);
    if ((i & 3) == 3) v = reduce(v, q, qinv);
  }
  if (h == 0) v += a.c0[t];
  out[o] = canon_full(v, q, qinv);
}
// out[h][t] = x[h][t] * c_t (mode 0), or out = x with c_t added to the first polynomial of
// every ciphertext (even h, mode 1), or out[h][t] = x[h][t] +/- y[h][t] (mode 2 add, mode 3
// subtract); x has xL limbs per polynomial (its first L read), y and out L
__global__ __launch_bounds__(256) void k_ct_elem(const double* __restrict__ x, const double* __restrict__ y,
                                                 double* __restrict__ out, ResArgs a,
                                                 const DevPrime* __restrict__ pr, int logn, int L, int xL, int mode,
                                                 size_t sx, size_t sy, size_t so) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y, h = blockIdx.z;
  const size_t ct = (size_t)(h >> 1), p = (size_t)(h & 1);
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = ct * so + (p * L + t) * n + k;
  double v = x[ct * sx + (p * xL + t) * n + k];
  if (mode == 0) v = mulc(v, a.c[t], a.cp[t], q);
  else if (mode == 1) v = p == 0 ? v + a.c[t] : v;
  else if (mode == 2) v = v + y[ct * sy + (p * L + t) * n + k];
  else v = v - y[ct * sy + (p * L + t) * n + k];
  out[o] = canon_full(v, q, qinv);
}

__global__ __launch_bounds__(256) void k_int_to_res(const int64_t* __restrict__ src, double* __restrict__ dst,
                                                    const DevPrime* __restrict__ pr, int logn, int nprimes) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y;
  const int p = blockIdx.z;
  const double q = pr[t].q, qinv = pr[t].qinv;
  dst[((size_t)p * nprimes + t) * n + k] = canon_full(int_residue(src[(size_t)p * n + k], q, qinv), q, qinv);
}

__global__ __launch_bounds__(256) void k_u64_to_res(const uint64_t* __restrict__ src, size_t words,
                                                    double* __restrict__ dst) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < words) dst[i] = (double)src[i];
}

__global__ __launch_bounds__(256) void k_res_to_u64(const double* __restrict__ src, size_t words,
                                                    uint64_t* __restrict__ dst) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < words) dst[i] = (uint64_t)src[i];
}

__global__ __launch_bounds__(256) void k_keygen_combine(double* __restrict__ key, const double* __restrict__ e,
                                                        const double* __restrict__ s,
                                                        const DevPrime* __restrict__ pr, int logn, int L, int np,
                                                        int alpha, uint32_t gal) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y;
  const int i = blockIdx.z;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const int lo = i * alpha, hi = min(lo + alpha, L);
  const double gad = (t >= lo && t < hi) ? pr[t].pmod : 0.0;
  const double a = key[(((size_t)i * 2 + 1) * np + t) * n + k];
  const double st = s[(size_t)t * n + k];
  const double sg = gal == 0u ? mul(st, st, q, qinv) : s[(size_t)t * n + perm((uint32_t)k, gal, logn)];
  const double ev = e[((size_t)i * np + t) * n + k];
  const double v = -mul(a, st, q, qinv) + ev + mul(gad, sg, q, qinv);
  key[(((size_t)i * 2 + 0) * np + t) * n + k] = canon_full(v, q, qinv);
}

__global__ __launch_bounds__(256) void k_enc_combine(double* __restrict__ ct, const double* __restrict__ v,
                                                     const double* __restrict__ s,
                                                     const DevPrime* __restrict__ pr, int logn, int L) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = (size_t)t * n + k;
  const double c1 = ct[(size_t)L * n + o];
  ct[o] = canon_full(v[o] - mul(c1, s[o], q, qinv), q, qinv);
}

__global__ __launch_bounds__(256) void k_dec_combine(const double* __restrict__ ct, double* __restrict__ out,
                                                     const double* __restrict__ s,
                                                     const DevPrime* __restrict__ pr, int logn, int L) {
  const int n = 1 << logn;
  const int k = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y;
  const double q = pr[t].q, qinv = pr[t].qinv;
  const size_t o = (size_t)t * n + k;
  out[o] = canon_full(ct[o] + mul(ct[(size_t)L * n + o], s[o], q, qinv), q, qinv);
}

}  // namespace

// ===========================================================================
// launchers
// ===========================================================================
// The library's fixed scratch array (fa_rotate_static): every GPU that loads
// the library holds its own copy.  The host refers to it only through the
// device address hipGetSymbolAddress returns on that GPU.
static __device__ __align__(256) double scratch[FA_STATIC_SCRATCH_BYTES / 8];

namespace fa {

// The address of `scratch` on `device` (which must be current), looked up once
// per device and kept; nullptr (with the HIP error in *err) if the lookup fails.
void* static_scratch(int device, hipError_t* err) {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static void* ptr[kMaxDev] = {};
  static hipError_t res[kMaxDev] = {};
  static bool done[kMaxDev] = {};
  if (device < 0 || device >= kMaxDev) {
    *err = hipErrorInvalidDevice;
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!done[device]) {
    void* p = nullptr;
    res[device] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    ptr[device] = res[device] == hipSuccess ? p : nullptr;
    done[device] = true;
  }
  *err = res[device];
  return ptr[device];
}

template <int SA>
static void launch_fwd(const fa_ctx* c, const LimbList& l, hipStream_t s) {
  using P = PassA<SA>;
  dim3 ga(c->n / P::TILE, l.n);
  hipLaunchKernelGGL(k_ntt_fwd_a<SA>, ga, dim3(256), 0, s, l, c->d_pr, c->d_twa_fwd);
  dim3 gb((c->n >> 8) / 16, l.n);
  hipLaunchKernelGGL(k_ntt_fwd_b, gb, dim3(256), 0, s, l, c->d_pr, c->d_twt_fwd, c->d_twr_fwd, c->logn);
}

template <int SA>
static void launch_inv(const fa_ctx* c, const LimbList& l, hipStream_t s) {
  using P = PassA<SA>;
  dim3 gb((c->n >> 8) / 16, l.n);
  hipLaunchKernelGGL(k_ntt_inv_b, gb, dim3(256), 0, s, l, c->d_pr, c->d_twt_inv, c->d_twr_inv, c->logn);
  dim3 ga(c->n / P::TILE, l.n);
  hipLaunchKernelGGL(k_ntt_inv_a<SA>, ga, dim3(256), 0, s, l, c->d_pr, c->d_twa_inv);
}

// rings above FA_SMALL_LOGN
#define FA_SA_SWITCH(fn, ...)            \
  switch (c->logn - 8) {                  \
    case 6: fn<6>(__VA_ARGS__); break;    \
    case 7: fn<7>(__VA_ARGS__); break;    \
    case 8: fn<8>(__VA_ARGS__); break;    \
    default: break;                       \
  }

void ntt_fwd(const fa_ctx* c, const LimbList& l, hipStream_t s) {
  if (l.n == 0) return;
  if (small_ring(c)) return sr_ntt(c, l, true, s);
  FA_SA_SWITCH(launch_fwd, c, l, s)
}

void ntt_inv(const fa_ctx* c, const LimbList& l, hipStream_t s) {
  if (l.n == 0) return;
  if (small_ring(c)) return sr_ntt(c, l, false, s);
  FA_SA_SWITCH(launch_inv, c, l, s)
}

void ntt_inv_b(const fa_ctx* c, const LimbList& l, hipStream_t s) {
  if (l.n == 0) return;
  dim3 gb((c->n >> 8) / 16, l.n);
  hipLaunchKernelGGL(k_ntt_inv_b, gb, dim3(256), 0, s, l, c->d_pr, c->d_twt_inv, c->d_twr_inv, c->logn);
}

static void strided(const fa_ctx* c, double* base, size_t stride, int count, int period, int prime_off,
                    hipStream_t s, bool fwd) {
  LimbBatch b(c, s, fwd);
  for (int i = 0; i < count; ++i) b.add(base + (size_t)i * stride, i % period + prime_off);
}

void ntt_fwd_strided(const fa_ctx* c, double* base, size_t stride, int count, int period, int prime_off,
                     hipStream_t s) {
  strided(c, base, stride, count, period, prime_off, s, true);
}
void ntt_inv_strided(const fa_ctx* c, double* base, size_t stride, int count, int period, int prime_off,
                     hipStream_t s) {
  strided(c, base, stride, count, period, prime_off, s, false);
}

// Target groups of a fused conversion launch: a launch of at least 256 workgroups
// (one per CU) keeps one group per source, as the repeated inverse passes of more
// cost more than they gain; a smaller one (one ciphertext) is split to about 256,
// at most one group per target.  Two workgroups fit a CU, but splitting to 512
// measured slower (rank reduction 2.22 against 2.19 ms, the face scan 6.41 against
// 6.26, one product at N=2^16 163 against 156 us, the fine level 817 against 788);
// 128 was between.
static int conv_groups(int wgs, int targets) {
  if (wgs >= 256) return 1;
  const int g = (256 + wgs - 1) / wgs;
  return g > targets ? targets : g;
}
template <int SA, int ALPHA>
static void launch_modup_fused(const fa_ctx* c, const MuArgs& a, int count, hipStream_t s) {
  using P = PassA<SA>;
  const int ngrp = conv_groups(c->n / P::TILE * c->dnum * count, c->np - ALPHA);
  dim3 g(c->n / P::TILE, c->dnum * ngrp, count);
  hipLaunchKernelGGL((k_modup_fused<SA, ALPHA>), g, dim3(512), 0, s, a, c->d_pr, c->d_twa_fwd, c->d_twa_inv,
                     c->d_mu_hat, c->d_mu_scale, c->logn, c->L, c->np, ngrp);
}
template <int SA>
static void launch_modup_fused_sa(const fa_ctx* c, const MuArgs& a, int count, hipStream_t s) {
  switch (c->alpha) {
    case 1: launch_modup_fused<SA, 1>(c, a, count, s); break;
    case 2: launch_modup_fused<SA, 2>(c, a, count, s); break;
    case 3: launch_modup_fused<SA, 3>(c, a, count, s); break;
    case 4: launch_modup_fused<SA, 4>(c, a, count, s); break;
    default: break;
  }
}

static void modup_pass_b(const fa_ctx* c, const MuItem* items, int count, hipStream_t s);

void modup_fused(const fa_ctx* c, const MuItem* items, int count, hipStream_t s, bool pass_b) {
  for (int off = 0; off < count; off += FA_MAXMU) {
    const int m = count - off < FA_MAXMU ? count - off : FA_MAXMU;
    MuArgs a;
    for (int i = 0; i < m; ++i) a.it[i] = items[off + i];
    FA_SA_SWITCH(launch_modup_fused_sa, c, a, m, s)
  }
  if (pass_b) modup_pass_b(c, items, count, s);
}

static void modup_pass_b(const fa_ctx* c, const MuItem* items, int count, hipStream_t s) {
  // second pass over every converted limb
  LimbList l;
  l.n = 0;
  dim3 gb((c->n >> 8) / 16, 0);
  auto flush = [&]() {
    if (!l.n) return;
    gb.y = l.n;
    hipLaunchKernelGGL(k_ntt_fwd_b, gb, dim3(256), 0, s, l, c->d_pr, c->d_twt_fwd, c->d_twr_fwd, c->logn);
    l.n = 0;
  };
  for (int b = 0; b < count; ++b)
    for (int i = 0; i < c->dnum; ++i) {
      const int lo = i * c->alpha, hi = lo + c->alpha < c->L ? lo + c->alpha : c->L;
      for (int t = 0; t < c->np; ++t) {
        if (t >= lo && t < hi) continue;
        l.ptr[l.n] = items[b].ext + ((size_t)i * c->np + t) * c->n;
        l.src[l.n] = l.ptr[l.n];
        l.prime[l.n] = t;
        l.scale[l.n] = 0.0;
        if (++l.n == FA_MAXL) flush();
      }
    }
  flush();
}

template <int SA, int KP>
static void launch_moddown_fused(const fa_ctx* c, const MdArgs& a, int count, hipStream_t s) {
  using P = PassA<SA>;
  const int ngrp = conv_groups(c->n / P::TILE * count, c->L);
  dim3 g(c->n / P::TILE, ngrp, count);
  hipLaunchKernelGGL((k_moddown_fused<SA, KP>), g, dim3(512), 0, s, a, c->d_pr, c->d_twa_fwd, c->d_twa_inv,
                     c->d_md_hat, c->d_md_scale, c->logn, c->L, ngrp);
}
template <int SA>
static void launch_moddown_fused_sa(const fa_ctx* c, const MdArgs& a, int count, hipStream_t s) {
  switch (c->K) {
    case 1: launch_moddown_fused<SA, 1>(c, a, count, s); break;
    case 2: launch_moddown_fused<SA, 2>(c, a, count, s); break;
    case 3: launch_moddown_fused<SA, 3>(c, a, count, s); break;
    case 4: launch_moddown_fused<SA, 4>(c, a, count, s); break;
    default: break;
  }
}

void moddown_fused(const fa_ctx* c, const MdItem* items, int count, hipStream_t s, bool pass_b) {
  for (int off = 0; off < count; off += FA_MAXMD) {
    const int m = count - off < FA_MAXMD ? count - off : FA_MAXMD;
    MdArgs a;
    for (int i = 0; i < m; ++i) a.it[i] = items[off + i];
    FA_SA_SWITCH(launch_moddown_fused_sa, c, a, m, s)
    if (!pass_b) continue;
    dim3 gb((c->n >> 8) / 16, c->L, m);
    hipLaunchKernelGGL(k_moddown_b, gb, dim3(256), 0, s, a, c->d_pr, c->d_twt_fwd, c->d_twr_fwd, c->logn);
  }
}


// 1-D grid of the key-switch kernels: nx * ny * ngroup work units, padded to
// whole groups of eight per query when nq > 1 (see ks_decode)
static unsigned ks_grid(int nx, int ny, int nq, int ngroup) {
  if (nq == 1) return 8u * ngroup * (((unsigned)nx * ny + 7) / 8);  // ks_decode_src
  const unsigned units = (unsigned)nx * ny * ngroup;
  return 8u * nq * ((units + 7) / 8);
}

// inverse of an odd Galois element modulo 2N (Newton's iteration modulo 2^32)
static uint32_t inv_galois(uint32_t g, int logn) {
  uint32_t x = g;
  for (int i = 0; i < 5; ++i) x *= 2u - g * x;
  return x & ((2u << logn) - 1u);
}

template <int DNUM>
static void launch_moddown_ks(const fa_ctx* c, const MdKsArgs& a, int m, int nq, hipStream_t s) {
  // eight 256-word rows per workgroup: twice the workgroups of sixteen-row tiles,
  // measured faster at 8 and 12 primes and even at 3
  const int ngroup = m / nq;
  dim3 gb(ks_grid((c->n >> 8) / 8, c->L, nq, ngroup));
  if (nq == 1)
    hipLaunchKernelGGL((k_moddown_ks_b<DNUM, 8, true>), gb, dim3(256), 0, s, a, c->d_pr, c->d_twt_fwd, c->d_twr_fwd,
                       c->logn, c->L, c->np, c->alpha, nq, ngroup);
  else
    hipLaunchKernelGGL((k_moddown_ks_b<DNUM, 8, false>), gb, dim3(256), 0, s, a, c->d_pr, c->d_twt_fwd,
                       c->d_twr_fwd, c->logn, c->L, c->np, c->alpha, nq, ngroup);
}

void moddown_ks(const fa_ctx* c, const MdKsItem* items, int count, hipStream_t s, int nq) {
  const int chunk = (FA_MAXMD / nq) * nq;
  for (int off = 0; off < count; off += chunk) {
    const int m = count - off < chunk ? count - off : chunk;
    MdKsArgs a;
    for (int i = 0; i < m; ++i) {
      a.it[i] = items[off + i];
      a.it[i].inv_gal = inv_galois(a.it[i].gal, c->logn);
    }
    switch (c->dnum) {
      case 1: launch_moddown_ks<1>(c, a, m, nq, s); break;
      case 2: launch_moddown_ks<2>(c, a, m, nq, s); break;
      case 3: launch_moddown_ks<3>(c, a, m, nq, s); break;
      case 4: launch_moddown_ks<4>(c, a, m, nq, s); break;
      case 5: launch_moddown_ks<5>(c, a, m, nq, s); break;
      case 6: launch_moddown_ks<6>(c, a, m, nq, s); break;
      case 7: launch_moddown_ks<7>(c, a, m, nq, s); break;
      case 8: launch_moddown_ks<8>(c, a, m, nq, s); break;
      default: break;
    }
  }
}

template <int DNUM>
static void launch_ks(const fa_ctx* c, const KsArgs& a, int m, hipStream_t s, int nq) {
  const int ngroup = m / nq;
  dim3 g(ks_grid(c->n / 256, c->K, nq, ngroup));
  hipLaunchKernelGGL(k_ks_inner<DNUM>, g, dim3(256), 0, s, a, c->d_pr, c->logn, c->L, c->np, nq, ngroup);
}

void ks_inner(const fa_ctx* c, const KsItem* items, int count, hipStream_t s, int nq) {
  const int chunk = (FA_MAXKS / nq) * nq;
  for (int off = 0; off < count; off += chunk) {
    KsArgs a;
    const int m = count - off < chunk ? count - off : chunk;
    for (int i = 0; i < m; ++i) {
      a.it[i] = items[off + i];
      a.it[i].inv_gal = inv_galois(a.it[i].gal, c->logn);
    }
    switch (c->dnum) {
      case 1: launch_ks<1>(c, a, m, s, nq); break;
      case 2: launch_ks<2>(c, a, m, s, nq); break;
      case 3: launch_ks<3>(c, a, m, s, nq); break;
      case 4: launch_ks<4>(c, a, m, s, nq); break;
      case 5: launch_ks<5>(c, a, m, s, nq); break;
      case 6: launch_ks<6>(c, a, m, s, nq); break;
      case 7: launch_ks<7>(c, a, m, s, nq); break;
      case 8: launch_ks<8>(c, a, m, s, nq); break;
      default: break;
    }
  }
}

template <int DNUM>
static void launch_ks_inv_b(const fa_ctx* c, const KsArgs& a, int m, hipStream_t s, int nq) {
  const int ngroup = m / nq;
  dim3 g(ks_grid(c->n >> 12, c->K, nq, ngroup));
  if (nq == 1)
    hipLaunchKernelGGL((k_ks_inv_b<DNUM, true>), g, dim3(256), 0, s, a, c->d_pr, c->d_twt_inv, c->d_twr_inv, c->logn,
                       c->L, c->np, nq, ngroup);
  else
    hipLaunchKernelGGL((k_ks_inv_b<DNUM, false>), g, dim3(256), 0, s, a, c->d_pr, c->d_twt_inv, c->d_twr_inv, c->logn,
                       c->L, c->np, nq, ngroup);
}

void ks_inv_b(const fa_ctx* c, const KsItem* items, int count, hipStream_t s, int nq) {
  if (c->dnum != 1) return;  // the host calls it for one-digit contexts only
  const int chunk = (FA_MAXKS / nq) * nq;
  for (int off = 0; off < count; off += chunk) {
    KsArgs a;
    const int m = count - off < chunk ? count - off : chunk;
    for (int i = 0; i < m; ++i) {
      a.it[i] = items[off + i];
      a.it[i].inv_gal = inv_galois(a.it[i].gal, c->logn);
    }
    launch_ks_inv_b<1>(c, a, m, s, nq);
  }
}

template <int DNUM>
static void launch_giant(const fa_ctx* c, const GiantArgs& a, int groups, hipStream_t s) {
  const int ntile = (c->n >> 8) / 16;
  const int rest8 = (ntile * c->np + 7) / 8;
  dim3 g((unsigned)(8 * a.nb * rest8), groups);
  hipLaunchKernelGGL((k_giant_ks<DNUM, 16>), g, dim3(256), 0, s, a, c->d_pr, c->d_twt_fwd, c->d_twr_fwd, c->logn,
                     c->L, c->np, c->alpha, ntile);
}

// Groups the giants of one launch are split into (see k_giant_ks): as many as
// keep the launch within the chip's 512 places, no more than there are giants,
// than the scratch holds or than k_sum_parts adds.
static int giant_groups(const fa_ctx* c, int nb, int ng, size_t part_words) {
  const long places = 512, wgs = (long)(c->n >> 12) * c->np * nb;
  const size_t one = (size_t)nb * 2 * c->np * c->n;
  long g = places / wgs;
  if (g > 1 + (long)(part_words / one)) g = 1 + (long)(part_words / one);
  if (g > ng) g = ng;
  return g < 1 ? 1 : g > 8 ? 8 : (int)g;
}

void giant_ks(const fa_ctx* c, const double* ext, const double* acc, size_t astride, const double* const* keys,
              const uint32_t* gals, int nb, int ng, double* u, double* part, size_t part_words, hipStream_t s) {
  const size_t ext_g = (size_t)c->dnum * c->np * c->n;
  for (int g0 = 0; g0 < ng; g0 += FA_MAXG) {
    GiantArgs a;
    const int m = ng - g0 < FA_MAXG ? ng - g0 : FA_MAXG;
    // chunks of giant indices: ext of chunk g0 is [nb][m] laid out inside [nb][ng]
    a.ext = ext + (size_t)g0 * ext_g;
    a.acc = acc;
    for (int g = 0; g < m; ++g) {
      a.key[g] = keys[g0 + g];
      a.gal[g] = gals[g0 + g];
    }
    a.u = u;
    a.part = part;
    a.astride = astride;
    a.nb = nb;
    a.ng = m;
    a.ngs = ng;
    a.g0 = 1 + g0;
    a.accumulate = g0 > 0;
    // a later chunk adds to u, so only a single one is split
    a.per = ng > FA_MAXG ? m : (m + giant_groups(c, nb, m, part_words) - 1) / giant_groups(c, nb, m, part_words);
    const int groups = (m + a.per - 1) / a.per;
    switch (c->dnum) {
      case 1: launch_giant<1>(c, a, groups, s); break;
      case 2: launch_giant<2>(c, a, groups, s); break;
      case 3: launch_giant<3>(c, a, groups, s); break;
      case 4: launch_giant<4>(c, a, groups, s); break;
      case 5: launch_giant<5>(c, a, groups, s); break;
      case 6: launch_giant<6>(c, a, groups, s); break;
      case 7: launch_giant<7>(c, a, groups, s); break;
      case 8: launch_giant<8>(c, a, groups, s); break;
      default: break;
    }
    if (groups > 1)
      hipLaunchKernelGGL(k_sum_parts, dim3(c->n / 256, nb * 2 * c->np), dim3(256), 0, s, u, part, groups - 1, c->d_pr,
                         c->logn, c->np);
  }
}

// Most (block, giant) accumulator pairs one pass keeps in registers for one
// query: 32 (default), 16 or 8; FA_MAC_PAIRS overrides it for tuning.  With
// NQ queries per pass the pairs per pass drop to 32 / NQ.
// the three-stage single-query kernel (FA_MAC_STAGES=2 selects the two-slot one)
// 17..31 pairs left: one padded 32-pair launch (FA_MAC_PAD=0: 16 + 16 / 8)
static bool mac_pad_wide() {
  static const bool v = [] {
    const char* e = getenv("FA_MAC_PAD");
    return !e || atoi(e) != 0;
  }();
  return v;
}
static bool mac_three_stages() {
  static const bool v = [] {
    const char* e = getenv("FA_MAC_STAGES");
    return !(e && atoi(e) == 2);
  }();
  return v;
}

// pairs per pass of a four-query group: 8 (default) or 16 (FA_MAC_Q4_PAIRS)
static int mac_q4_pairs() {
  static const int v = [] {
    const char* e = getenv("FA_MAC_Q4_PAIRS");
    return e && atoi(e) == 16 ? 16 : 8;
  }();
  return v;
}

static int mac_pairs_max() {
  static const int v = [] {
    const char* e = getenv("FA_MAC_PAIRS");
    const int r = e ? atoi(e) : 32;
    return (r == 8 || r == 16) ? r : 32;
  }();
  return v;
}

// ring depth of the staged loads: as many slots as fit beside the other
// workgroup sharing a CU's 160 KB of LDS (two slots at one query x 32 pairs)
template <int NQ, int NACC>
struct MacStages {
  static constexpr int BYTES = 4 * (NACC + 2 * NQ) * 64 * 8;
  static constexpr int S = BYTES * 3 <= 80 * 1024 ? 3 : 2;
};

template <int NQ, int NACC>
static void launch_mac(MacArgs a, int nchunk, const fa_ctx* c, hipStream_t s) {
  a.ntile = (int)((size_t)c->L * c->n / 256);
  a.nchunk = nchunk;
  const unsigned grid = nchunk == 1 ? (unsigned)a.ntile : 8u * nchunk * ((a.ntile + 7) / 8);
  if constexpr (NQ == 1) {
    if (mac_three_stages())
      hipLaunchKernelGGL((k_mac_diag3<NACC>), dim3(grid), dim3(256), 0, s, a, c->d_pr, c->logn);
    else
      hipLaunchKernelGGL((k_mac_diag<NQ, NACC, MacStages<NQ, NACC>::S>), dim3(grid), dim3(256), 0, s, a, c->d_pr,
                         c->logn);
  } else {
    hipLaunchKernelGGL((k_mac_diag<NQ, NACC, MacStages<NQ, NACC>::S>), dim3(grid), dim3(256), 0, s, a, c->d_pr,
                       c->logn);
  }
}

// pairs p0.. of the current query group: all full chunks of the group's widest
// pass in one launch, then one narrower launch for the rest
template <int NQ, int WIDE>
static int mac_chunks(MacArgs& a, int p0, const fa_ctx* c, hipStream_t s) {
  const int left = a.n_pairs - p0;
  a.pair0 = p0;
  if (left >= WIDE) {
    launch_mac<NQ, WIDE>(a, left / WIDE, c, s);
    return p0 + (left / WIDE) * WIDE;
  }
  if (NQ == 1 && WIDE == 32 && left > 16 && mac_pad_wide()) {
    // one padded launch: the missing pairs re-read the last pair's rows (cache
    // hits) instead of a second launch re-reading every rotated query
    launch_mac<NQ, WIDE>(a, 1, c, s);
    return p0 + WIDE;
  }
  if (WIDE > 16 && left > 8) {
    launch_mac<NQ, (WIDE > 16 ? 16 : WIDE)>(a, 1, c, s);
    return p0 + 16;
  }
  launch_mac<NQ, 8>(a, 1, c, s);
  return p0 + 8;
}

void mac_diag(const fa_ctx* c, const double* const* q, const double* const* qrot, int nq,
              const double* const* blocks, int n_blocks, int B, int G, double* const* acc, hipStream_t s) {
  const int pmax = mac_pairs_max();
  int logG = 0;
  while ((1 << logG) < G) ++logG;
  const size_t ctw = (size_t)2 * c->L * c->n;
  for (int j0 = 0; j0 < nq;) {
    const int m = nq - j0 >= 4 ? 4 : nq - j0 >= 2 ? 2 : 1;  // queries sharing this plaintext pass
    for (int b0 = 0; b0 < n_blocks; b0 += FA_MAXBLK) {
      const int nb = n_blocks - b0 < FA_MAXBLK ? n_blocks - b0 : FA_MAXBLK;
      MacArgs a;
      for (int j = 0; j < m; ++j) {
        a.q0[j] = q[j0 + j];
        a.qrot[j] = qrot[j0 + j];
        a.acc[j] = acc[j0 + j] + (size_t)b0 * G * ctw;
      }
      for (int i = 0; i < nb; ++i) a.blk[i] = blocks[b0 + i];
      a.n_pairs = nb * G;
      a.B = B;
      a.logG = logG;
      a.L = c->L;
      for (int p0 = 0; p0 < a.n_pairs;) {
        if (m == 4) p0 = mac_q4_pairs() == 16 ? mac_chunks<4, 16>(a, p0, c, s) : mac_chunks<4, 8>(a, p0, c, s);
        else if (m == 2) p0 = pmax >= 32 ? mac_chunks<2, 16>(a, p0, c, s) : mac_chunks<2, 8>(a, p0, c, s);
        else if (pmax >= 32) p0 = mac_chunks<1, 32>(a, p0, c, s);
        else if (pmax >= 16) p0 = mac_chunks<1, 16>(a, p0, c, s);
        else p0 = mac_chunks<1, 8>(a, p0, c, s);
      }
    }
    j0 += m;
  }
}

template <int NACC>
static void launch_mac_ct(MacCtArgs a, int nchunk, const fa_ctx* c, hipStream_t s) {
  a.ntile = (int)((size_t)c->L * c->n / 256);
  a.nchunk = nchunk;
  const unsigned grid = nchunk == 1 ? (unsigned)a.ntile : 8u * nchunk * ((a.ntile + 7) / 8);
  hipLaunchKernelGGL((k_mac_diag_ct<NACC>), dim3(grid), dim3(256), 0, s, a, c->d_pr, c->logn);
}

void mac_diag_ct(const fa_ctx* c, const double* q, const double* qrot, const double* const* blocks, int n_blocks,
                 int B, int G, double* acc, hipStream_t s) {
  int logG = 0;
  while ((1 << logG) < G) ++logG;
  const size_t ln = (size_t)c->L * c->n;
  for (int b0 = 0; b0 < n_blocks; b0 += FA_MAXBLK) {
    const int nb = n_blocks - b0 < FA_MAXBLK ? n_blocks - b0 : FA_MAXBLK;
    MacCtArgs a;
    a.q0 = q;
    a.qrot = qrot;
    a.acc = acc + (size_t)b0 * G * 3 * ln;
    for (int i = 0; i < nb; ++i) a.blk[i] = blocks[b0 + i];
    a.n_pairs = nb * G;
    a.B = B;
    a.logG = logG;
    a.L = c->L;
    for (int p0 = 0; p0 < a.n_pairs;) {
      const int left = a.n_pairs - p0;
      a.pair0 = p0;
      if (left >= 16) {
        launch_mac_ct<16>(a, left / 16, c, s);
        p0 += (left / 16) * 16;
      } else {
        launch_mac_ct<8>(a, 1, c, s);
        p0 += 8;
      }
    }
  }
}

void mul_plain(const fa_ctx* c, const double* ct, const double* const* pts, int count, double* out, hipStream_t s) {
  for (int off = 0; off < count; off += FA_MAXPT) {
    PtArgs a;
    const int m = count - off < FA_MAXPT ? count - off : FA_MAXPT;
    for (int i = 0; i < m; ++i) a.pt[i] = pts[off + i];
    dim3 g((unsigned)((size_t)c->L * c->n / 256), m);
    hipLaunchKernelGGL(k_mul_plain, g, dim3(256), 0, s, ct, a, out + (size_t)off * 2 * c->L * c->n, c->d_pr,
                       c->logn, c->L);
  }
}

static ResArgs res_args(const fa_ctx* c, const uint64_t* cres, int L) {
  ResArgs a;
  for (int t = 0; t < FA_MAXLIMB; ++t) {
    a.c[t] = t < L ? (double)cres[t] : 0.0;
    a.cp[t] = t < L ? a.c[t] / (double)c->primes[t] : 0.0;
  }
  return a;
}

template <int SA>
static void launch_rescale_fused(const fa_ctx* c, const double* last, double* lift, int n_polys, hipStream_t s) {
  using P = PassA<SA>;
  const int ngrp = conv_groups(c->n / P::TILE * n_polys, c->L - 1);
  hipLaunchKernelGGL(k_rescale_fused<SA>, dim3(c->n / P::TILE, ngrp, n_polys), dim3(512), 0, s, last, lift, c->d_pr,
                     c->d_twa_fwd, c->d_twa_inv, c->L, ngrp);
}

// The last limb's inverse, its centred lift and the forward transform to the
// other primes share their passes as in ModDown: three launches (a row pass, the
// columns of both transforms with the lift between, a row pass that also
// combines) for six.
void rescale(const fa_ctx* c, const double* ct, int n_polys, double* out, double* scratch, hipStream_t s) {
  const size_t n = c->n;
  const int L = c->L;
  double* last = scratch;                        // [n_polys][N]
  double* lift = scratch + (size_t)n_polys * n;  // [n_polys][L-1][N]
  {
    LimbBatch inv(c, s, false, !small_ring(c));
    for (int h = 0; h < n_polys; ++h) inv.add(last + (size_t)h * n, L - 1, ct + ((size_t)h * L + L - 1) * n);
  }
  std::vector<uint64_t> inv(L - 1);
  const uint64_t qlast = c->primes[L - 1];
  for (int t = 0; t < L - 1; ++t) {
    const uint64_t q = c->primes[t];
    // (q_last mod q)^(q-2) mod q
    unsigned __int128 b = qlast % q, r = 1;
    for (uint64_t e = q - 2; e; e >>= 1) {
      if (e & 1) r = r * b % q;
      b = b * b % q;
    }
    inv[t] = (uint64_t)r;
  }
  if (small_ring(c)) {
    SrRes r{};
    for (int t = 0; t < L - 1; ++t) r.c[t] = (double)inv[t];
    return sr_rescale(c, ct, last, n_polys, out, r, s);
  }
  FA_SA_SWITCH(launch_rescale_fused, c, last, lift, n_polys, s)
  hipLaunchKernelGGL(k_rescale_b, dim3((c->n >> 8) / 16, L - 1, n_polys), dim3(256), 0, s, ct, lift, out,
                     res_args(c, inv.data(), L - 1), c->d_pr, c->d_twt_fwd, c->d_twr_fwd, c->logn, L);
}

void tensor(const fa_ctx* c, const double* x, int xL, size_t sx, const double* y, int yL, size_t sy, int count,
            double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_tensor, dim3(c->n / 256, c->L, count), dim3(256), 0, s, x, y, out, c->d_pr, c->logn, c->L,
                     xL, yL, sx, sy);
}

void tensor_list(const fa_ctx* c, const double* const* xs, const int* xLs, const double* const* ys, const int* yLs,
                 int count, double* out, hipStream_t s) {
  const size_t step = (size_t)3 * c->L * c->n;
  for (int j0 = 0; j0 < count; j0 += FA_MAXTERM) {
    const int m = std::min(FA_MAXTERM, count - j0);
    TensorList a{};
    for (int j = 0; j < m; ++j) {
      a.x[j] = xs[j0 + j];
      a.y[j] = ys[j0 + j];
      a.xL[j] = xLs[j0 + j];
      a.yL[j] = yLs[j0 + j];
    }
    hipLaunchKernelGGL(k_tensor_list, dim3(c->n / 256, c->L, m), dim3(256), 0, s, a, out + (size_t)j0 * step,
                       c->d_pr, c->logn, c->L);
  }
}

void cheb_fix(const fa_ctx* c, double* prod, int count, const double* t1, int t1L, const uint64_t* const* cres,
              const int* odd, hipStream_t s) {
  const size_t step = (size_t)2 * c->L * c->n;
  for (int j0 = 0; j0 < count; j0 += FA_MAXTERM) {
    const int m = std::min(FA_MAXTERM, count - j0);
    ChebFixArgs a{};
    for (int j = 0; j < m; ++j) {
      const ResArgs r = res_args(c, cres[j0 + j], c->L);
      for (int t = 0; t < FA_MAXLIMB; ++t) {
        a.c[j][t] = r.c[t];
        a.cp[j][t] = r.cp[t];
      }
      a.odd[j] = odd[j0 + j];
    }
    hipLaunchKernelGGL(k_cheb_fix, dim3(c->n / 256, c->L, 2 * m), dim3(256), 0, s, prod + (size_t)j0 * step,
                       t1, a, c->d_pr, c->logn, c->L, t1L);
  }
}

void lincomb(const fa_ctx* c, double* out, const double* const* xs, const int* xLs, const uint64_t* const* cres,
             int nterm, const uint64_t* c0res, hipStream_t s) {
  for (int i0 = 0; i0 < nterm; i0 += FA_MAXTERM) {
    const int m = std::min(FA_MAXTERM, nterm - i0);
    LinArgs a{};
    for (int i = 0; i < m; ++i) {
      const ResArgs r = res_args(c, cres[i0 + i], c->L);
      a.x[i] = xs[i0 + i];
      a.xL[i] = xLs[i0 + i];
      for (int t = 0; t < FA_MAXLIMB; ++t) {
        a.c[i][t] = r.c[t];
        a.cp[i][t] = r.cp[t];
      }
    }
    if (i0 == 0 && c0res)
      for (int t = 0; t < c->L; ++t) a.c0[t] = (double)c0res[t];
    a.nterm = m;
    a.accumulate = i0 > 0;
    hipLaunchKernelGGL(k_lincomb, dim3(c->n / 256, c->L, 2), dim3(256), 0, s, out, a, c->d_pr, c->logn, c->L);
  }
}

void ct_elem(const fa_ctx* c, const double* x, const double* y, double* out, int n_polys, const uint64_t* cres,
             int mode, hipStream_t s, int xL, size_t sx, size_t sy, size_t so) {
  std::vector<uint64_t> zero(c->L, 0);
  const int xl = xL ? xL : c->L;
  const size_t n = c->n, ctw = 2 * (size_t)c->L * n;
  // the defaults: consecutive ciphertexts (x with xl limbs per polynomial)
  if (sx == (size_t)-1) sx = 2 * (size_t)xl * n;
  if (sy == (size_t)-1) sy = ctw;
  if (so == (size_t)-1) so = ctw;
  hipLaunchKernelGGL(k_ct_elem, dim3(c->n / 256, c->L, n_polys), dim3(256), 0, s, x, y, out,
                     res_args(c, cres ? cres : zero.data(), c->L), c->d_pr, c->logn, c->L, xl, mode, sx, sy, so);
}

void add_limbs(const fa_ctx* c, double* dst, const double* src, int n_limbs, int period, hipStream_t s) {
  dim3 g(c->n / 256, n_limbs);
  hipLaunchKernelGGL(k_add_limbs, g, dim3(256), 0, s, dst, src, c->d_pr, c->logn, period);
}

void int_to_res(const fa_ctx* c, const int64_t* src, int n_polys, int nprimes, double* dst, hipStream_t s) {
  for (int p0 = 0; p0 < n_polys; p0 += 65535) {
    const int m = n_polys - p0 < 65535 ? n_polys - p0 : 65535;
    dim3 g(c->n / 256, nprimes, m);
    hipLaunchKernelGGL(k_int_to_res, g, dim3(256), 0, s, src + (size_t)p0 * c->n,
                       dst + (size_t)p0 * nprimes * c->n, c->d_pr, c->logn, nprimes);
  }
}

template <int SA>
static void launch_fwd_a_int(const fa_ctx* c, const int64_t* src, int count, double* dst, hipStream_t s) {
  using P = PassA<SA>;
  hipLaunchKernelGGL(k_ntt_fwd_a_int<SA>, dim3(c->n / P::TILE, c->L, count), dim3(256), 0, s, src, dst, c->d_pr,
                     c->d_twa_fwd, c->L);
}
void int_to_ntt(const fa_ctx* c, const int64_t* src, int count, double* dst, hipStream_t s) {
  if (small_ring(c)) {
    int_to_res(c, src, count, c->L, dst, s);
    return ntt_fwd_strided(c, dst, c->n, count * c->L, c->L, 0, s);
  }
  FA_SA_SWITCH(launch_fwd_a_int, c, src, count, dst, s)
  LimbList l;
  l.n = 0;
  for (int i = 0; i < count * c->L; ++i) {
    l.ptr[l.n] = dst + (size_t)i * c->n;
    l.src[l.n] = l.ptr[l.n];
    l.prime[l.n] = i % c->L;
    l.scale[l.n] = 0.0;
    if (++l.n == FA_MAXL || i == count * c->L - 1) {
      hipLaunchKernelGGL(k_ntt_fwd_b, dim3((c->n >> 8) / 16, l.n), dim3(256), 0, s, l, c->d_pr, c->d_twt_fwd,
                         c->d_twr_fwd, c->logn);
      l.n = 0;
    }
  }
}

void u64_to_res(const uint64_t* src, size_t words, double* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_u64_to_res, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, src, words, dst);
}

void res_to_u64(const double* src, size_t words, uint64_t* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_res_to_u64, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, src, words, dst);
}

void keygen_combine(const fa_ctx* c, double* key, const double* e_ntt, uint32_t gal, hipStream_t s) {
  dim3 g(c->n / 256, c->np, c->dnum);
  hipLaunchKernelGGL(k_keygen_combine, g, dim3(256), 0, s, key, e_ntt, c->d_s, c->d_pr, c->logn, c->L, c->np,
                     c->alpha, gal);
}

void enc_combine(const fa_ctx* c, double* ct, const double* v, hipStream_t s) {
  dim3 g(c->n / 256, c->L);
  hipLaunchKernelGGL(k_enc_combine, g, dim3(256), 0, s, ct, v, c->d_s, c->d_pr, c->logn, c->L);
}

void dec_combine(const fa_ctx* c, const double* ct, double* out, hipStream_t s) {
  dim3 g(c->n / 256, c->L);
  hipLaunchKernelGGL(k_dec_combine, g, dim3(256), 0, s, ct, out, c->d_s, c->d_pr, c->logn, c->L);
}

}  // namespace fa
