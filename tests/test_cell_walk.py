"""The index walk of the neighbour scan on the CPU: every candidate of the 27
cells once, also where the walk stops and goes on, and no entry read behind the sorted particles' spare ones, where the
16 particles of a wave have ranges of very different lengths.  (The scan drops
what lies past a particle's range, so results cannot show such a read.)"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import systems

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_15508_amd", "csrc")

DRIVER = r"""
#include "cell_walk.hpp"
using namespace dplr::mlp;
extern "C" int scan_pad() { return kScanPad; }
// start [ncells + 1], cell [n][3] of the sorted particles; listed[i]: candidates
// of particle i.  Returns the largest entry read.
extern "C" int walk(int n, const int* nc, const int* start, const int* cell, long* listed) {
  int most = 0;
  for (int i0 = 0; i0 < n; i0 += 16) {
    CellWalk w[16];
    bool ends = false;
    for (int p = 0; p < 16; ++p) {
      const int i = i0 + p < n ? i0 + p : n - 1;
      w[p] = CellWalk{start, nc[0], nc[1], nc[2], cell[3 * i], cell[3 * i + 1], cell[3 * i + 2], i0 + p < n, 0, 0, 0, 0};
      ends = ends || w[p].at_end();
    }
    const int dq = ends ? 1 : 2;
    int q = 0, chunk = 0;
    auto read = [&]() {  // lanes g < kDescLanes, loads u < kScan: j0 + g + kDescLanes u
      for (int p = 0; p < 16; ++p) {
        const int last = w[p].j0 + (kDescLanes - 1) + kDescLanes * (kScan - 1);
        if (w[p].j0 < 0) return false;
        if (last > most) most = last;
      }
      return true;
    };
    for (int p = 0; p < 16; ++p) w[p].begin(0, 0, dq);
    if (!read()) return -1;
    while (q < kSegments) {
      bool more = false;
      for (int p = 0; p < 16; ++p) {
        if (i0 + p < n) listed[i0 + p] += w[p].left();
        else if (w[p].left()) return -2;
        w[p].advance();
        more = more || w[p].j0 < w[p].j1;
      }
      ++chunk;
      if (!more) {
        q += dq;
        chunk = 0;
        for (int p = 0; p < 16; ++p) w[p].next_segment(q + dq);
      }
      if (!read()) return -1;
      // a scan that stopped here goes on from the same place
      for (int p = 0; p < 16 && q < kSegments; ++p) {
        CellWalk r = w[p];
        r.begin(q, chunk, dq);
        if (r.j0 != w[p].j0 || r.j1 != w[p].j1 || r.j0n != w[p].j0n || r.j1n != w[p].j1n) return -3;
      }
    }
  }
  return most;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("walk")
    (d / "walk.cpp").write_text(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(d / "walk.cpp"), "-o",
                    str(d / "walk.so")], check=True, capture_output=True, timeout=120)
    return ctypes.CDLL(str(d / "walk.so"))


def _uniform(rng, n, box):
    return rng.random((n, 3)) * box


def _slab(rng, n, box):  # a dense slab below the top face, vapour elsewhere
    pos = rng.random((n, 3)) * box
    k = n - n // 20
    pos[:k, 2] = box[2] * (0.85 + 0.15 * rng.random(k))
    return pos


def _droplet(rng, n, box):  # ... and a droplet in the last corner's cells
    k = n - n // 20
    pos = rng.random((n, 3)) * box
    pos[:k] = np.mod(box * (1.0 - 1e-3) - np.abs(rng.normal(0.0, 2.0, (k, 3))), box)
    return pos


def _water(name, seed=0):
    if name == "box":
        s = systems.training_box(seed)
    else:
        s = systems.workload(1).system()
    return s.all_pos(), np.asarray(s.box, dtype=float)


@pytest.mark.parametrize("kind,n,box", [
    ("water", 0, None), ("box", 0, None),
    (_uniform, 1, (12.0, 12.0, 12.0)), (_uniform, 17, (12.5, 40.0, 13.0)), (_uniform, 1000, (12.5, 12.5, 12.5)),
    (_uniform, 20000, (40.0, 52.0, 60.0)), (_slab, 4000, (30.0, 24.0, 50.0)), (_droplet, 6000, (40.0, 40.0, 40.0)),
])
def test_walk_reads_the_candidates_and_stays_inside(lib, kind, n, box):
    if callable(kind):
        box = np.array(box)
        pos = kind(np.random.default_rng(n), n, box)
    else:
        pos, box = _water(kind)
    n = len(pos)
    nc = np.floor(box / 4.0).astype(np.int32)
    c = np.clip((np.mod(pos, box) / box * nc).astype(np.int64), 0, nc - 1)
    flat = (c[:, 2] * nc[1] + c[:, 1]) * nc[0] + c[:, 0]
    order = np.argsort(flat, kind="stable")
    cell = np.ascontiguousarray(c[order], dtype=np.int32)
    count = np.bincount(flat, minlength=int(nc.prod()))
    start = np.concatenate([[0], np.cumsum(count)]).astype(np.int32)
    listed = np.zeros(n, dtype=np.int64)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    most = lib.walk(n, ptr(nc), ptr(start), ptr(cell), ptr(listed))
    assert most >= 0
    grid = count.reshape(nc[2], nc[1], nc[0])
    around = sum(np.roll(grid, (a, b, d), (0, 1, 2)) for a in (-1, 0, 1) for b in (-1, 0, 1) for d in (-1, 0, 1))
    assert np.array_equal(listed, around[cell[:, 2], cell[:, 1], cell[:, 0]])
    print(f"largest entry read: n + {most - n}")
    assert most < n + lib.scan_pad()
