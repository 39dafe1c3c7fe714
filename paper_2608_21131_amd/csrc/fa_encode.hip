// Float encoding of enrollment on the GPU: the slots of many plaintexts at once
// to integer coefficients,
//   m_k = rint(scale (2/N) sum_j v_j cos(pi k 5^j / N)),
// by the length-N transform of fa_encode (fa_host.cpp: encode_one).  Every
// butterfly is the same float64 operations on the same table values as there, so
// the coefficients are the same integers; only the order between independent
// butterflies differs.
//
// On the host one block of 128 diagonals at N = 2^15 took 7.5 ms on 16 threads.
// Here it is two passes over 16 B a coefficient: stages of span 2..256 on runs of
// 256 words (k_enc_a, which gathers the slots from the rows itself), the others on
// columns (k_enc_b).  A tile of 4,096 points lives in LDS and goes through it once
// per stage.  Of the block's 329 us of kernels these two take 68 and 66; the
// residues of 8 primes (rounding to residues and their transform, 8 L bytes a
// coefficient, three times) take the other 195.

#include <hip/hip_runtime.h>

#include "fa_internal.h"

namespace {

constexpr int kTile = 4096;  // points of a workgroup's tile (32 KB for each part)

// the slot values of plaintext p (see the encoders in fa.h)
struct Rows {
  fa::EncArgs a;
  int S;
  __device__ double operator()(int p, int s) const {
    if (a.kind == fa::ENC_ROWS) {
      const int row = p * (S / a.d) + s / a.d, u = s % a.d;
      return row < a.n_rows && u < a.dim ? (double)a.rows[(size_t)row * a.dim + u] : 0.0;
    }
    const int i = (s - (p / a.B) * a.B) & (S - 1);  // pre-rotated right by the giant step
    if (a.kind == fa::ENC_DIAG) {
      const int col = (i + p) & (a.d - 1);
      return i < a.n_rows && col < a.dim ? (double)a.rows[(size_t)i * a.dim + col] : 0.0;
    }
    return (double)a.rows[(size_t)((i + p) & (a.n_rows - 1)) * a.d + (i & (a.d - 1))];  // n_rows = d_in
  }
};

// (ur, ui) +- (vr, vi) w in place
__device__ __forceinline__ void bfly(double* re, double* im, int iu, int iv, double wr, double wi) {
  const double br = re[iv], bi = im[iv], ur = re[iu], ui = im[iu];
  const double vr = br * wr - bi * wi, vi = br * wi + bi * wr;
  re[iu] = ur + vr;
  im[iu] = ui + vi;
  re[iv] = ur - vr;
  im[iv] = ui - vi;
}

// stages of span 2..256 on 256-word runs of the bit-reversed input; z_p at
// z + p * zst: real parts [N], then imaginary [N]
__global__ __launch_bounds__(256) void k_enc_a(Rows v, int p0, double* __restrict__ z, size_t zst,
                                               const double2* __restrict__ root, const uint32_t* __restrict__ slot,
                                               int logn) {
  __shared__ double re[kTile], im[kTile];
  const int n = 1 << logn, len0 = n < kTile ? n : kTile;
  const int base = blockIdx.x * kTile, p = blockIdx.y;
  for (int e = threadIdx.x; e < len0; e += 256) {
    re[e] = v(p0 + p, (int)slot[__brev((uint32_t)(base + e)) >> (32 - logn)]);
    im[e] = 0.0;
  }
  __syncthreads();
  for (int s = 0; s < 8; ++s) {
    const int h = 1 << s;
    for (int b = threadIdx.x; b < len0 / 2; b += 256) {
      const int j = b & (h - 1), iu = ((b >> s) << (s + 1)) + j;
      const double2 w = root[(size_t)j << (logn - s - 1)];
      bfly(re, im, iu, iu + h, w.x, w.y);
    }
    __syncthreads();
  }
  double* zr = z + p * zst + base;
  for (int e = threadIdx.x; e < len0; e += 256) {
    zr[e] = re[e];
    zr[n + e] = im[e];
  }
}

// the stages of span 512..N on columns, the twist and the rounding: m_k, and
// INT64_MIN where the value is no number or out of range (as the host's cast)
__global__ __launch_bounds__(256) void k_enc_b(const double* __restrict__ z, size_t zst, int64_t* __restrict__ out,
                                               const double2* __restrict__ root, const double2* __restrict__ twist,
                                               int logn, double scale) {
  __shared__ double re[kTile], im[kTile];
  const int n = 1 << logn, rows = n >> 8, sa = logn - 8;
  const int cols = rows > 16 ? kTile / rows : 256, lc = __ffs(cols) - 1;
  const int c0 = blockIdx.x * cols, p = blockIdx.y;
  const int total = rows << lc;
  const double* zr = z + p * zst;
  for (int e = threadIdx.x; e < total; e += 256) {
    const int k = ((e >> lc) << 8) + c0 + (e & (cols - 1));
    re[e] = zr[k];
    im[e] = zr[n + k];
  }
  __syncthreads();
  for (int s = 0; s < sa; ++s) {
    const int h = 1 << s;
    for (int b = threadIdx.x; b < total / 2; b += 256) {
      const int c = b & (cols - 1), r = b >> lc, j = r & (h - 1);
      const int iu = ((((r >> s) << (s + 1)) + j) << lc) + c;
      const double2 w = root[(size_t)((j << 8) + c0 + c) << (sa - s - 1)];
      bfly(re, im, iu, iu + (h << lc), w.x, w.y);
    }
    __syncthreads();
  }
  const double ninv = 1.0 / (double)n;  // a power of two: the product is the quotient
  for (int e = threadIdx.x; e < total; e += 256) {
    const int k = ((e >> lc) << 8) + c0 + (e & (cols - 1));
    const double2 t = twist[k];
    const double x = rint(scale * (re[e] * t.x + im[e] * t.y) * ninv);
    out[(size_t)p * n + k] = fabs(x) < 0x1p63 ? (int64_t)x : INT64_MIN;
  }
}

}  // namespace

namespace fa {

void encode_slots(const fa_ctx* c, const EncArgs& a, int p0, int count, double* z, size_t zst, int64_t* out,
                  double scale, hipStream_t s) {
  const int tiles = c->n > kTile ? c->n / kTile : 1;
  const double2* root = reinterpret_cast<const double2*>(c->d_fft);
  const double2* twist = root + c->n / 2;
  const uint32_t* slot = reinterpret_cast<const uint32_t*>(twist + c->n);
  hipLaunchKernelGGL(k_enc_a, dim3(tiles, count), dim3(256), 0, s, Rows{a, c->n / 2}, p0, z, zst, root, slot,
                     c->logn);
  hipLaunchKernelGGL(k_enc_b, dim3(tiles, count), dim3(256), 0, s, z, zst, out, root, twist, c->logn, scale);
}

}  // namespace fa
