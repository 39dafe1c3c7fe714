"""The residue arithmetic's stated bounds, on the CPU: the giant steps' digit sums stay exact at the
largest products that row-pass words and key words can give, for one to eight digits."""
import os
import subprocess

from oracle import ckks

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# what fa_arith.h takes from the HIP header, with the same rounding
HIP_STAND_IN = """#pragma once
#include <cmath>
#include <cstdint>
#define __device__
#define __forceinline__ inline
using std::rint;
inline double __fma_rn(double a, double b, double c) { return std::fma(a, b, c); }
inline uint32_t __brev(uint32_t x) {
  uint32_t r = 0;
  for (int i = 0; i < 32; ++i) r |= ((x >> i) & 1u) << (31 - i);
  return r;
}
"""


def test_digit_sums_are_exact_at_their_bounds(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP_STAND_IN)
    exe = str(tmp_path / "arith_bounds")
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", str(tmp_path), "-I",
                        os.path.join(ROOT, "paper_2608_21131_amd", "csrc"), os.path.join(ROOT, "tests", "arith_bounds.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    primes = [q for logn in (14, 16) for q in ckks.Params(logn=logn, L=16, K=4).primes]
    r = subprocess.run([exe], input="\n".join(map(str, primes)), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
    assert r.stdout.split() == [w for q in primes for w in ("ok", str(q))]
