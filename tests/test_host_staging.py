"""The device staging that fa_encrypt, fa_decrypt and fa_export_coeffs share, on the CPU: whichever
HIP call of a pass fails, the call returns FA_E_HIP with nothing left queued on the staging."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CLANG = "/opt/rocm/lib/llvm/bin/clang++"


@pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG)), reason="ROCm compilers not installed")
def test_failed_calls_leave_no_work_on_the_staging(tmp_path):
    inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2608_21131_amd", "csrc")]
    objs = []
    for src in (os.path.join(ROOT, "paper_2608_21131_amd", "csrc", "fa_host.cpp"),
                os.path.join(ROOT, "tests", "host_staging.cpp")):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        r = subprocess.run([HIPCC, "--offload-host-only", "-c", "-O1", "-std=c++17", "-ffp-contract=off", *inc, src,
                            "-o", obj], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        objs.append(obj)
    exe = str(tmp_path / "host_staging")
    # no HIP runtime: the stand-ins are the only ones called
    r = subprocess.run([CLANG, *objs, "-Wl,--unresolved-symbols=ignore-all", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert [ln.split()[:2] for ln in r.stdout.splitlines()] == [["ok", k] for k in ("encrypt", "decrypt", "export")]
