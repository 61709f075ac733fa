"""Order of the 64-slot tile's workgroups, compiled for the host: every piece of every block once, and an even share of the
work for each of the 8 XCDs also where experts with many rows follow one another."""
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_16214_amd", "csrc")
MAIN = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <cstdio>
#include <cstdlib>
#include "mid_order.hpp"
int main(int argc, char** argv) {       // nblk, nwork, capacity in blocks: xcd, block, piece of every workgroup that has one
  const int nblk = atoi(argv[1]), nwork = atoi(argv[2]);
  const long long grid = moe::mid_grid(atoll(argv[3]), nwork);
  for (long long pid = 0; pid < grid; ++pid) {
    int b = -1, w = -1;
    if (moe::mid_work((int)pid, nblk, nwork, b, w)) printf("%d %d %d\n", (int)pid & 7, b, w);
  }
}
"""


@pytest.fixture(scope="module")
def order(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("order")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "order")], check=True)

    def run(nblk, nwork, capacity):
        out = subprocess.run([str(d / "order"), str(nblk), str(nwork), str(capacity)], check=True, capture_output=True).stdout
        return np.array(out.split(), dtype=np.int64).reshape(-1, 3)
    return run


@pytest.mark.parametrize("nblk", [0, 1, 7, 8, 17, 31, 32, 33, 63, 64, 67, 127, 128, 131, 300])
def test_every_piece_once(order, nblk):
    for nwork in (1, 2, 3, 7, 8, 9, 16, 56, 112):
        for capacity in (nblk, nblk + 5):
            w = order(nblk, nwork, capacity)
            assert w.shape[0] == nblk * nwork
            got = w[:, 1] * nwork + w[:, 2]
            assert np.array_equal(np.sort(got), np.arange(nblk * nwork)) and (w[:, 2] < nwork).all()


@pytest.mark.parametrize("E,avg,power", [(8, 20, 2.4), (8, 20, 1.0), (32, 20, 1.0), (64, 12, 1.0), (128, 16, 1.0), (256, 10, 1.0), (256, 10, 2.4), (256, 22, 0.0)])
def test_the_xcds_share_the_work_evenly(order, E, avg, power):
    """Rows by rank ** -power, capped as top-k routing caps them (an expert has a token once); a block costs its live
    16-row parts plus one for its weights.  In runs of blocks the busiest XCD had up to 1.9 times the mean."""
    share = np.arange(1, E + 1) ** -power
    rows = np.minimum(avg * E * share / share.sum(), avg * E / 2).round().astype(int)
    cost = np.array([1 + -(-min(64, r - at) // 16) for r in rows for at in range(0, r, 64)])
    w = order(cost.size, 56, cost.size)
    per_xcd = np.bincount(w[:, 0], weights=cost[w[:, 1]], minlength=8)
    assert per_xcd.max() <= 1.15 * per_xcd.mean()
