"""The rules that size launches, compiled for the host: what they choose has to
fit the buffers for every size and build constant, not for the default ones
alone."""
import ctypes
import os
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
    so.sort_chunk.argtypes = [ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_long]
    return so


@pytest.mark.parametrize("max_chunks", [1, 2, 7, 15, 16, 17, 100, 256])
def test_sort_chunks_fit_the_histograms(lib, max_chunks):
    for n in [1, 255, 256, 257, 1024, 1025, 4096, 4097, 8191, 16383, 16384, 16385, 65537, 288768, 2 ** 31 - 1]:
        for nbins in (1, 4096, 4097, 16384):
            c = lib.sort_chunk(n, nbins, max_chunks, 256)
            assert c > 0 and c % 256 == 0
            assert -(-n // c) <= max_chunks, (n, nbins)
