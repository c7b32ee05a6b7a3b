"""The addresses of the quantized GEMM of the comparison and linear layers, enumerated on the CPU: the
kernel and this check share the arithmetic (csrc/wq_direct_walk.h), so an access that would leave a
caller's buffer is found without a GPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_request_of_the_quantized_gemm_leaves_its_buffer(tmp_path):
    exe = tmp_path / "walk"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2412_19867_amd", "csrc"),
                    os.path.join(ROOT, "tests", "direct_walk_check.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
