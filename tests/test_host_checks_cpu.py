"""Host-side C++ checks of the tiles' preparation and of the kernels' index
arithmetic, built with g++ and the sanitizers (no GPU code); see the sources
under tests/host_cpp/."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_07628_amd", "csrc")


def run_check(tmp_path, prog, *flags):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / prog)
    subprocess.run([gxx, "-O1", "-std=c++17", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    *flags, os.path.join(ROOT, "tests", "host_cpp", prog + ".cpp"),
                    os.path.join(CSRC, "dpdlp_host.cpp"), "-o", exe, "-lpthread"],
                   check=True, timeout=300)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-2000:]
    assert out.stdout.strip().endswith("ok")


def test_walks_end_at_the_largest_positions(tmp_path):
    run_check(tmp_path, "walk_check")


@pytest.mark.parametrize("nnz_max,segs_max", [(2048, 1024), (1000, 300), (4096, 1024), (5000, 4096)])
def test_tile_kernel_holds_every_tile_size(tmp_path, nnz_max, segs_max):
    run_check(tmp_path, "tile_limits_check", f"-DDPDLP_TILE_NNZ_MAX={nnz_max}",
              f"-DDPDLP_TILE_SEGS_MAX={segs_max}")


def test_merged_splits_keep_their_order_and_fill_the_chip(tmp_path):
    run_check(tmp_path, "merge_check")
