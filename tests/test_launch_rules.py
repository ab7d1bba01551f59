"""The rules that size launches, compiled for the host: what they choose has to
fit the buffers for every size and build constant, not for the default ones
alone."""
import ctypes
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_15508_amd", "csrc")

DRIVER = r"""
#include "launch_rules.hpp"
extern "C" long sort_chunk(long n, int nbins, int max_chunks, long align) {
  return dplr::sort_chunk(n, nbins, max_chunks, align);
}
extern "C" int plane_threads(long pts, int spread, int most) {
  return spread ? dplr::fused_spread_threads(pts, most) : dplr::fused_inverse_threads(pts, most);
}
extern "C" int z_threads(long points, long blocks, int most) { return dplr::fused_z_threads(points, blocks, most); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(d / "rules.cpp"), "-o",
                    str(d / "rules.so")], check=True, capture_output=True, timeout=120)
    so = ctypes.CDLL(str(d / "rules.so"))
    so.sort_chunk.restype = ctypes.c_long
    so.plane_threads.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int]
    so.z_threads.argtypes = [ctypes.c_long, ctypes.c_long, ctypes.c_int]
    so.sort_chunk.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_long]
    return so


@pytest.mark.parametrize("max_chunks", [1, 2, 7, 15, 16, 17, 100, 256])
def test_sort_chunks_fit_the_histograms(lib, max_chunks):
    for n in [1, 255, 256, 257, 1024, 1025, 4096, 4097, 8191, 16383, 16384, 16385, 65537, 288768, 2 ** 31 - 1]:
        for nbins in (1, 4096, 4097, 16384):
            c = lib.sort_chunk(n, nbins, max_chunks, 256)
            assert c > 0 and c % 256 == 0
            assert -(-n // c) <= max_chunks, (n, nbins)


def _kernel_constants():
    src = open(os.path.join(CSRC, "mixed_radix_kernels.hpp")).read()
    num = lambda pat: int(re.search(pat, src).group(1))
    return num(r"kFusedZMaxPts = (\d+)"), num(r"kFusedZThreads = (\d+)")


def test_fused_blocks_hold_their_points(lib):
    # points a thread: 128 KiB of complex values over 768 (FP32) or 512 (FP64)
    # threads; blocks of whole waves, within the launch bounds
    for most, cap in ((768, 16384), (512, 8192)):
        per = -(-cap // most)
        for spread in (0, 1):
            for pts in range(4, cap + 1):
                t = lib.plane_threads(pts, spread, most)
                assert t % 64 == 0 and 64 <= t <= most and pts <= per * t
                assert not spread or t >= 512
    cap, most = _kernel_constants()
    for points in range(2, cap + 1):
        for blocks in (1, 1024, 1025, 10 ** 5):
            t = lib.z_threads(points, blocks, most)
            assert t % 64 == 0 and 64 <= t <= most and points <= cap // most * t
            if blocks <= 1024:  # few blocks: no thread has two points while there are threads for them
                assert t == most or t >= points
