// Error paths of the client calls that share the context's device staging, on the
// CPU: tests/test_host_staging.py links this file with the library's host source.
// The HIP calls and kernel launchers it needs are stand-ins below: copies only count
// as queued until the stream is synchronised, and the k-th HIP call of a pass fails.
// Whatever fails, a call must not return with work queued that uses the staging: the
// next caller, on another stream, takes the same memory.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "fa_internal.h"

static int queued = 0;    // copies and launches since the last synchronisation
static int calls = 0;     // failable calls of this pass
static int fail_at = -1;  // the call that fails

static hipError_t step() { return calls++ == fail_at ? hipErrorUnknown : hipSuccess; }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
  const hipError_t e = step();
  if (e == hipSuccess) ++queued;
  return e;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  queued = 0;
  return hipSuccess;
}
hipError_t hipGetLastError() { return step(); }
const char* hipGetErrorString(hipError_t) { return "injected"; }
}

namespace fa {
void u64_to_res(const uint64_t*, size_t, double*, hipStream_t) { ++queued; }
void res_to_u64(const double*, size_t, uint64_t*, hipStream_t) { ++queued; }
void int_to_res(const fa_ctx*, const int64_t*, int, int, double*, hipStream_t) { ++queued; }
void ntt_fwd_strided(const fa_ctx*, double*, size_t, int, int, int, hipStream_t) { ++queued; }
void ntt_inv_strided(const fa_ctx*, double*, size_t, int, int, int, hipStream_t) { ++queued; }
void enc_combine(const fa_ctx*, double*, const double*, hipStream_t) { ++queued; }
void dec_combine(const fa_ctx*, const double*, double*, hipStream_t) { ++queued; }
}  // namespace fa

int main() {
  fa_ctx c;
  c.logn = 10;
  c.n = 1 << c.logn;
  c.L = 2;
  c.np = 3;
  const size_t n = c.n, L = c.L;
  std::vector<double> dev(2 * L * n + 32);
  fa_buf ct{};
  ct.dev = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(dev.data()) + 255) & ~uintptr_t(255));
  ct.bytes = 2 * L * n * 8;
  std::vector<int64_t> m(n), e(n);
  std::vector<uint64_t> a(L * n), res(2 * L * n);
  auto encrypt = [&] { return fa_encrypt(&c, m.data(), 40, a.data(), e.data(), &ct, nullptr); };
  auto decrypt = [&] { return fa_decrypt(&c, &ct, res.data(), nullptr); };
  auto exports = [&] { return fa_export_coeffs(&c, &ct, res.data(), nullptr); };
  auto check = [&](const char* name, auto call) {
    fail_at = -1;
    calls = 0;
    if (call() != FA_OK || queued) {
      std::printf("%s: fails or leaves work queued without an injected error: %s\n", name, fa_last_error());
      return false;
    }
    const int total = calls;
    if (total < 2) return false;
    for (fail_at = 0; fail_at < total; ++fail_at) {
      calls = 0;
      const int rc = call();
      if (rc != FA_E_HIP) {
        std::printf("%s: call %d failed, returned %d\n", name, fail_at, rc);
        return false;
      }
      if (queued) {
        std::printf("%s: call %d failed, %d queued at return\n", name, fail_at, queued);
        return false;
      }
      if (!c.export_mu.try_lock()) return false;
      c.export_mu.unlock();
    }
    std::printf("ok %s %d\n", name, total);
    return true;
  };
  const bool r0 = check("encrypt", encrypt), r1 = check("decrypt", decrypt), r2 = check("export", exports);
  return r0 && r1 && r2 ? 0 : 1;
}
