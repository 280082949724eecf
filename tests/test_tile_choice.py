"""The tile choice of a lone GEMM launch (csrc/gemm_tiles.h, host code) for the
problems of the GPU tests that are meant to run on each tile."""
import os
import shutil
import subprocess

import pytest

from tests.test_gpu_kernels import LONE_TILES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def choice(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("needs g++ and the ROCm headers")
    exe = str(tmp_path_factory.mktemp("tiles") / "tile_check")
    cmd = [gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "paper_2206_04959_amd", "csrc"),
           os.path.join(ROOT, "tests", "sanitize", "tile_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def run(problems):
        args = [",".join(str(int(v)) for v in p) for p in problems]
        return subprocess.run([exe, *args], capture_output=True, text=True, check=True).stdout.split()
    return run


def test_gpu_test_shapes_reach_their_tiles(choice):
    assert choice([(*mnk, 0) for mnk in LONE_TILES]) == list(LONE_TILES.values())
    for mnk, tile, transposed in zip(LONE_TILES, LONE_TILES.values(), choice([(*mnk, 1) for mnk in LONE_TILES])):
        assert transposed == tile if tile != "64x128" else transposed != "64x128", mnk


def test_large_problems_take_large_tiles(choice):
    assert choice([(4096, 4096, 4096, 0), (4096, 3072, 3072, 0)]) == ["256x256", "256x192"]
