"""Which workgroup of the fused kernel works on which block, enumerated on the CPU: the kernel, its launch and this
check share the arithmetic (csrc/wq_fused_blocks.h)."""
import os
import subprocess

import pytest

from test_fused_rounds_gpu import BANDS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("blocks") / "blocks"
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2412_19867_amd", "csrc"),
                    os.path.join(ROOT, "tests", "fused_blocks_check.cpp"), "-o", str(exe)], check=True)
    return lambda *a: subprocess.run([str(exe), *map(str, a)], capture_output=True, text=True)


def test_every_block_has_one_workgroup(check):
    r = check()
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("shape,mode,one,four", BANDS, ids=lambda v: "%dx%dx%d_%d-%d_F%d_g%d" % v if isinstance(v, tuple) and len(v) == 7 else str(v))
def test_the_banded_layers_of_the_gpu_tests_have_a_narrower_last_band(check, wq, shape, mode, one, four):
    L = wq.Plan(*shape).layout
    for nt, (band, last) in ((1, one), (2, four)):
        assert check(L.T_pad, L.Cout_pad, L.Cin, L.n, nt, nt).stdout.split() == [str(mode), str(band), str(last)]
