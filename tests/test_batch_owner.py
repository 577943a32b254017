"""A batch's outcomes own their results (host only, built with g++ against the
library)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1807_07691_amd")


def test_dropped_outcomes_free_their_results(tmp_path):
    import paper_1807_07691_amd  # noqa: F401  (the library is built)
    exe = str(tmp_path / "owner")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           os.path.join(ROOT, "tests", "native", "batch_owner_check.cpp"),
                           os.path.join(PKG, "libgsmat.so"), "-Wl,-rpath," + PKG, "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
