"""The block GEMM whose loaders deal a stage to 256 threads refuses eight waves when it is compiled; what other classes
inherit from it does not."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_12949_amd", "csrc")
USE = """
#include "ffuse_gemm0.h"
typedef ffuse::FirstGemm<__bf16, false, 128, 128, 2, %d> Gemm;
__global__ void kernel(const void* p, int n) {
    __shared__ __attribute__((aligned(16))) char smem[Gemm::LDS_BYTES];
    Gemm::Ctx c;
    ffuse::f32x16 acc[Gemm::HT][Gemm::MT], acc3[1][1];
    %s
    Gemm::store_tile_rt(0, acc, acc3, smem, 8, 0, 0, 1, 1, (int)threadIdx.x);
}
"""
CALLS = {"init_a": "Gemm::init_a(c, p, n, 0, 0, n, n, (int)threadIdx.x);",
         "init_b": "Gemm::init_b(c, p, p, n, n, n, 0, (int)threadIdx.x);",
         "run": "Gemm::run(smem, c, 0, n, acc, acc3, (int)threadIdx.x);",
         "run_deep": "Gemm::run_deep(smem, c, 0, n, acc, acc3, (int)threadIdx.x);"}


def _compile(tmp_path, waves, call):
    src = tmp_path / "use.hip"
    src.write_text(USE % (waves // 2, call))
    return subprocess.run(["hipcc", "-x", "hip", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only", "-fsyntax-only", "-w",
                           "-I", CSRC, str(src)], capture_output=True, text=True)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
@pytest.mark.parametrize("name", sorted(CALLS))
def test_own_loaders_are_for_four_waves(name, tmp_path):
    r = _compile(tmp_path, 4, CALLS[name])
    assert r.returncode == 0, r.stderr
    r = _compile(tmp_path, 8, CALLS[name])
    assert r.returncode != 0 and "loaders are for four waves" in r.stderr, r.stderr


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_the_inherited_part_takes_eight(tmp_path):
    r = _compile(tmp_path, 8, "")
    assert r.returncode == 0, r.stderr
